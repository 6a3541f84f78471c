// The fused CG kernel with the whole state of an inner solve on the chip.
//
// Same method as k_fused_cg (Chronopoulos-Gear CG on A_s d = r_s, one
// reduction per iteration, then u_s += d), laid out so that a CG iteration
// moves next to nothing through the caches:
//  * a thread owns one pair of x-neighbours, the vertex (even closure index)
//    and the mid-point after it, over all planes of its block's z-range, so
//    r, w, s, p and x are private to the thread: r and s stay in registers
//    (the plane loop is unrolled over the P planes a block may hold), p and x
//    in LDS, w in LDS (WL) or, where LDS is full, in a private buffer that
//    the L2 cache holds;
//  * a wave owns whole rows of pairs, one idle lane between them, so the x-pass
//    takes its neighbours from the adjacent lanes (DPP) instead of LDS and
//    only the operand plane is shared: one workgroup barrier per plane;
//  * a mid-point row has no +-2 entries and constant centres, so half of the
//    nodes need three taps along x and no coefficients of their own;
//  * a team of blocks shares a subdomain as in k_fused_cg, and exchanges only w
//    on the two edge planes each side: every member carries r and s of its
//    halo planes along itself. Blocks are persistent: a team takes subdomains
//    from the work-ordered list until none is left.
//
// What bounds it: the latency of a sweep's chain, no longer memory. A sweep is its
// own planes, one barrier each, whose vector instructions (about 90 per pair and
// plane, three waves per SIMD at 33 x 33 nodes) are the larger part of them; the
// neighbours' halo planes, one or two a side; and the meeting, two trips between
// compute units and the wait for the slowest member. Cycles of one block, from its own
// clock: at 33 x 33 nodes 1,460 to 1,550 a plane, 1,940
// with second-order terms, 2,510 where w is in the private buffer too; 1,700 to 3,100
// for a neighbour's halo planes; 6,400 to 14,000 for the meeting. So 64^3 elements in
// 64 subdomains, in fours, spend 11,700 of 29,300 cycles a sweep on their own planes,
// 128^3 in 512, in threes, 21,300 of 32,700. At 17 x 17 nodes in teams of eight it is
// 2,900 of 11,900, the meeting 7,000. In FP64 a plane takes 6,200 (registers spill).
//
// Whole solves against k_fused_cg, each in the shape that the tuner finds best for it,
// on one GPU: 128^3 elements in 512 subdomains, second-order condition, 1633 -> 1009
// ms; 96^3 in 216, 985 -> 914; 64^3 in 64, 701 -> 669; 16^3 in 4, 69.2 -> 64.3; 37 x 29
// x 23 in 27 uneven, 17.6 -> 17.0; 48^3 in 27, FP64 and adjoint, 767 -> 381.
// k_fused_cg stays where a plane has few rows and many subdomains fill the chip
// anyway: a block of six waves leaves no room for a second one on its unit
// (256 columns of 12 x 12 x 96 nodes: 427 ms there, 694 here; 64 slabs of 11 x 39
// x 639: 290 against 297), and where whole subdomains in one block need no team at all
// (256 of 32^3: 123 against 132 ms).
#pragma once

#include "sos_device.h"
#include "sos_mail.h"

namespace sos {

// ---------------------------------------------------------------------------- lane exchange

// Value of the lane below (CTRL 0x138, wave_shr:1) or above (0x130,
// wave_shl:1); 0 at the end of the wave.
template <int CTRL>
__device__ __forceinline__ int dpp0(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, true);
}
template <int CTRL>
__device__ __forceinline__ float lane_move(float v) {
  return __int_as_float(dpp0<CTRL>(__float_as_int(v)));
}
template <int CTRL>
__device__ __forceinline__ double lane_move(double v) {
  return __hiloint2double(dpp0<CTRL>(__double2hiint(v)), dpp0<CTRL>(__double2loint(v)));
}
template <typename T>
__device__ __forceinline__ T from_below(T v) { return lane_move<0x138>(v); }
template <typename T>
__device__ __forceinline__ T from_above(T v) { return lane_move<0x130>(v); }

// A value that is the same in every lane, moved to scalar registers. (Without
// the empty asm the compiler folds the builtin away where it knows the value to
// be uniform, and keeps what the vector unit computed in vector registers. The
// builtin, not the instruction in asm: the compiler then adds the wait states
// that the instruction needs after a vector write of its source.)
__device__ __forceinline__ int uniform(int v) {
  asm("" : "+v"(v));
  return __builtin_amdgcn_readfirstlane(v);
}
__device__ __forceinline__ float uniform(float v) { return __int_as_float(uniform(__float_as_int(v))); }
__device__ __forceinline__ double uniform(double v) {
  return __hiloint2double(uniform(__double2hiint(v)), uniform(__double2loint(v)));
}
// v + D for a scalar v, a sum that the compiler does not see through.
template <int D>
__device__ __forceinline__ int scalar_add(int v) {
  int r;
  asm("s_add_i32 %0, %1, %2" : "=s"(r) : "s"(v), "i"(D) : "scc");
  return r;
}
// Either value, both at hand (a conditional between variables that a functor
// holds by reference would select their addresses and keep them in scratch).
template <typename T>
__device__ __forceinline__ T pick(bool c, T a, T b) { return c ? a : b; }

// ---------------------------------------------------------------------------- types

template <typename T>
struct alignas(2 * sizeof(T)) P2 {
  T a, b;  // the pair's vertex and mid-point
};
template <typename T>
struct alignas(4 * sizeof(T) > 16 ? 16 : 4 * sizeof(T)) P4 {
  T a, b, c, d;
};

// A pair on its way to another block: 64-bit words of 32 bits of data and the
// sender's 32-bit sequence number, written and read with agent-scope atomics
// (see team_sum), each word whole or not at all. The reader knows from the
// words themselves that they have arrived, so neither side waits for stores
// to complete before a flag.
template <typename T>
constexpr int mail_words = 2 * (int)sizeof(T) / 4;
__device__ __forceinline__ unsigned long long mail_word(unsigned v, unsigned seq) {
  return (unsigned long long)v | ((unsigned long long)seq << 32);
}
__device__ __forceinline__ void mail_write(unsigned long long* p, unsigned seq, float a, float b) {
  st_coh(p, mail_word(__float_as_uint(a), seq));
  st_coh(p + 1, mail_word(__float_as_uint(b), seq));
}
__device__ __forceinline__ void mail_write(unsigned long long* p, unsigned seq, double a, double b) {
  st_coh(p, mail_word((unsigned)__double2loint(a), seq));
  st_coh(p + 1, mail_word((unsigned)__double2hiint(a), seq));
  st_coh(p + 2, mail_word((unsigned)__double2loint(b), seq));
  st_coh(p + 3, mail_word((unsigned)__double2hiint(b), seq));
}
// Reads a pair; true once all its words carry seq.
__device__ __forceinline__ bool mail_read(const unsigned long long* p, unsigned seq, P2<float>& v) {
  const unsigned long long a = ld_coh(p), b = ld_coh(p + 1);
  v.a = __uint_as_float((unsigned)a);
  v.b = __uint_as_float((unsigned)b);
  return (unsigned)(a >> 32) == seq && (unsigned)(b >> 32) == seq;
}
__device__ __forceinline__ bool mail_read(const unsigned long long* p, unsigned seq, P2<double>& v) {
  const unsigned long long a = ld_coh(p), b = ld_coh(p + 1), c = ld_coh(p + 2), d = ld_coh(p + 3);
  v.a = __hiloint2double((int)(unsigned)b, (int)(unsigned)a);
  v.b = __hiloint2double((int)(unsigned)d, (int)(unsigned)c);
  return (unsigned)(a >> 32) == seq && (unsigned)(b >> 32) == seq && (unsigned)(c >> 32) == seq &&
         (unsigned)(d >> 32) == seq;
}

// LDS by its own 32-bit address: constant offsets then go into the instruction.
__device__ __forceinline__ uint32_t lds_address(const void* p) {
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void*)p;
}
template <typename V>
__device__ __forceinline__ V& lds_at(uint32_t o) {
  return *(V*)(__attribute__((address_space(3))) V*)(uintptr_t)o;
}

template <int I, int N, class F>
__device__ __forceinline__ void unroll(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>());
    unroll<I + 1, N>(f);
  }
}

// ---------------------------------------------------------------------------- reduction

// Sum N values over the block and its team (the tagged slots of team_sum; the
// partials carry their own tag and nothing else is ordered by them), one pass:
// wave sums, then one wave adds them, publishes, waits for the members
// and adds theirs. Every thread receives the sums. The block's last wave, which
// owns no rows, does this while meanwhile() runs on the others: both wait for
// other blocks, and in one wave the second wait would follow the first. ticks:
// the longest wait for a member.
constexpr int kChipSums = 3;
struct ChipRed {
  double wave[kChipSums * 16];
  double total[kChipSums];
  int fail;
  int job;
};

// Partial sums of subdomain s: [member][parity][kTeamSlot], TM members.
__device__ __forceinline__ double* chip_part(const FusedArgs& a, int s) {
  return a.team_part + (size_t)s * a.team * 2 * kTeamSlot;
}

template <int N, class F>
__device__ __forceinline__ void chip_sum(double (&v)[N], ChipRed& sh, const FusedArgs& a, int s, int tau, int TM,
                                         int epoch, unsigned long long ticks, int& fail, F&& meanwhile) {
  static_assert(N <= kChipSums, "a row of lanes per sum");
  // (opaque, so that no address below is kept in registers through the sweep)
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int lane = tid & 63, w = uniform(tid >> 6), nw = blockDim.x >> 6;
#pragma unroll
  for (int n = 0; n < N; ++n) v[n] = wave_sum63(v[n]);
  if (lane == 63) {
#pragma unroll
    for (int n = 0; n < N; ++n) sh.wave[n * 16 + w] = v[n];
  }
  if (tid == 0) sh.fail = 0;
  __syncthreads();
  if (w == nw - 1) {
    // row n of the lanes adds the waves' parts of sum n, then the members',
    // sixteen at a time
    const int n = lane >> 4, m = lane & 15;
    double part = row_sum15(n < N && m < nw ? sh.wave[n * 16 + m] : 0.0);
    if (TM > 1) {
      double* const base = chip_part(a, s) + (epoch & 1) * kTeamSlot + n;
      const unsigned tag = (unsigned)((epoch + 1) & 0xFF);
      const unsigned want = (unsigned)((epoch + 1 + a.tag_skew) & 0xFF);
      if (n < N && m == 15) st_coh(base + (size_t)tau * 2 * kTeamSlot, with_tag(part, tag));
      part = 0.0;
      const unsigned long long t0 = wall_clock64();
      for (int mm = m; mm < TM; mm += 16) {
        if (n >= N) break;
        const double* q = base + (size_t)mm * 2 * kTeamSlot;
        double val = ld_coh(q);
        while (tag_of(val) != want) {
          if (wall_clock64() - t0 > ticks) {
            sh.fail = 1;
            break;
          }
          val = ld_coh(q);
        }
        part += with_tag(val, 0u);
      }
      part = row_sum15(part);
    }
    if (n < N && m == 15) sh.total[n] = part;
  } else if (meanwhile()) {
    sh.fail = 1;
  }
  __syncthreads();
#pragma unroll
  for (int n = 0; n < N; ++n) v[n] = sh.total[n];
  // (the flag is cleared again before the next meeting's first barrier, after
  // the barriers of a whole sweep)
  if (TM > 1) fail |= sh.fail;
}

// ---------------------------------------------------------------------------- kernel

// P: most planes of a block's z-range; Q: second-order face terms; WL: w in LDS.
// The number of pairs per row is each subdomain's own. As a compile-time constant (17
// of them, subdomains 16 elements wide) it puts the offsets of neighbouring rows
// into the instructions, but up to sixteen more registers spill. Whole solves with and
// without it: 128^3 in 512 992 against 1011 ms, 96^3 in 216 922 against 914, 48^3 in
// 27 in FP64 392 against 382, 32 copies of 32^3 133 against 132.
// From 13 planes on a thread's registers hold r alone: s takes x's place in LDS
// and x goes to private memory, read and written every second sweep only (two
// steps along p at once, in the order of the single ones).
template <typename T, int P, bool Q, bool WL>
__global__ void __launch_bounds__(kChipThreads) k_chip_cg(Dev d, const int32_t* __restrict__ bfirst, FusedArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ ChipRed sh;
  const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
  const int TM = a.team;
  // Teams form from the blocks as they start (one ticket each), never from
  // block indices: a member waits only for blocks that are running or next in
  // line, so a grid that shares the GPU with other kernels cannot lock up.
  int ticket = blockIdx.x;
  if (TM > 1) {
    if (tid == 0) sh.job = atomicAdd(&a.queue[0], 1);
    __syncthreads();
    ticket = uniform(sh.job);
    __syncthreads();
  }
  const int team = uniform(ticket / TM), tau = ticket - team * TM;
  if (team >= a.n_teams) return;  // (the host launches n_teams teams)
  int job = team;
  // sequence number of the sweep: the same in every member, another in every
  // sweep since the mailboxes were cleared
  unsigned seq = mail_first((unsigned)uniform(a.queue[2]), a.chip_span);
  unsigned long long ticks = a.spin_ticks * 64ull;  // the first meeting: a member may still wait for a place
  while (job < a.n_jobs) {
    const int s = uniform(a.fmap[job].s);
    const SubDesc& sd = d.subs[s];
    const int nx = uniform(sd.n[0]), ny = uniform(sd.n[1]), nz = uniform(sd.n[2]);
    const int zb0 = uniform((tau * nz) / TM), zb1 = uniform(((tau + 1) * nz) / TM), zlen = zb1 - zb0;
    const int xk = uniform(sd.klo[0]), yk = uniform(sd.klo[1]), zk = uniform(sd.klo[2]);
    const int np = chip_pairs(nx, xk);
    const int R = chip_rows(np);
    const int nslots = np * ny;
    const int rq = lane / (np + 1), e = lane - rq * (np + 1);
    const int row = wave * R + rq;
    const bool live = rq < R && e < np && row < ny;
    const int slot = live ? row * np + e : 0;
    const int ia = 2 * e - xk, ib = ia + 1;  // local x index of the two nodes
    const bool la = live && ia >= 0 && ia < nx, lb = live && ib < nx;
    const int S = nx * ny;
    const int64_t off = sd.off;
    // LDS: w (WL), p and x, the two operand planes. A read of one plane past
    // a private array's end (the prefetch) stays inside.
    const int zmax = (nz + TM - 1) / TM;
    P2<T>* const wl = reinterpret_cast<P2<T>*>(smem);
    P4<T>* const px = reinterpret_cast<P4<T>*>(smem + (WL ? chip_even((size_t)zmax * nslots) * sizeof(P2<T>) : 0));
    P2<T>* const opl = reinterpret_cast<P2<T>*>(px + (size_t)zmax * nslots);
    const int opn = np * (ny + 4);
    constexpr bool XG = P > 12;  // x in private memory, s in LDS
    int brk = 0, t = 0, epoch = 0, tfail = 0;
    T xstep = T(0);  // step along p that x does not hold yet
    P2<T>* const xg = reinterpret_cast<P2<T>*>(a.chip_x) + (size_t)ticket * (P + kChipAhead) * blockDim.x;
    if (zmax > P || (TM > 1 && nz < 2 * TM) || R < 1 ||
        (ny + R - 1) / R >= (int)(blockDim.x >> 6) || chip_lds(np, ny, zmax, sizeof(T), WL) > a.lds_bytes ||
        nslots > a.chip_slots)
      brk |= kBrkLaunch;  // (the host sizes the launch for every subdomain)
    double rb[2];
    part_sums<1>(a.res_part, bfirst[s], bfirst[s + 1], rb);
    const double rr = rb[0], bb = rb[1];
    const double stop2 =
        uniform(fmax(uniform(a.tol_rel * a.tol_rel) * rr, uniform(a.tol_abs * a.tol_abs) * bb));
    // the inner solve runs on sig r, sig a power of two (see k_fused_cg)
    int sexp = 0;
    if (isfinite(rr) && rr > 0.0) {
      int e2 = 0;
      (void)frexp(rr / double(nx * ny * nz), &e2);
      sexp = min(max(-(e2 / 2), -100), 100);
    }
    sexp = uniform(sexp);
    const double stop2s = uniform(stop2 * ldexp(1.0, 2 * sexp));
    if (!isfinite(rr) || !isfinite(bb)) brk |= kBrkNonFinite;
    if (!brk && rr > stop2 && a.max_inner > 0) {
      // ------------------------------------------------ coefficients
      const T ksx = uniform(T(sd.ks[0])), msx = uniform(T(sd.ms[0]));
      const T zks = uniform(T(sd.ks[2])), zms = uniform(T(sd.ms[2]));
      const T zelo = uniform(T(sd.elo[2])), zehi = uniform(T(sd.ehi[2]));
      const int zne2 = uniform(sd.ne2[2]);
      // uniform entries of the 1D rows, in scalar registers (the z centres by
      // row kind: mid-point, vertex, lower and upper end)
      const T kx1 = uniform(T(-8) * ksx), mx1 = uniform(T(2) * msx), kxb = uniform(T(16) * ksx),
              mxb = uniform(T(16) * msx);
      const T kz1 = uniform(T(-8) * zks), mz1 = uniform(T(2) * zms);
      const T kzm = uniform(T(16) * zks), kzv = uniform(T(14) * zks), kzl = uniform(T(7) * zks + zelo),
              kzh = uniform(T(7) * zks + zehi);
      const T mzm = uniform(T(16) * zms), mzv = uniform(T(8) * zms), mze = uniform(T(4) * zms);
      const Row<T> rx = row_of<T>(2 * e, uniform(sd.ne2[0]), ksx, msx, T(sd.elo[0]), T(sd.ehi[0]));
      const T kxa = rx.k0, mxa = rx.m0;
      const T ksy = T(sd.ks[1]), msy = T(sd.ms[1]);
      const Row<T> ry = row_of<T>(row + yk, uniform(sd.ne2[1]), ksy, msy, T(sd.elo[1]), T(sd.ehi[1]));
      // an idle lane's row is zero, and so is everything it hands its neighbours
      const T ky0 = live ? ry.k0 : T(0), my0 = live ? ry.m0 : T(0), ky2 = live ? ry.k2 : T(0),
              my2 = live ? ry.m2 : T(0), ky1 = live ? T(-8) * ksy : T(0), my1 = live ? T(2) * msy : T(0);
      T exa = T(0), ey = T(0), qxa = T(0), qy = T(0), zqlo = T(0), zqhi = T(0);
      if constexpr (Q) {
        const bool x0 = e == 0, x1 = 2 * e == sd.ne2[0];  // an x end is a vertex
        const bool y0 = row + yk == 0, y1 = row + yk == sd.ne2[1];
        exa = x0 ? T(sd.elo[0]) : (x1 ? T(sd.ehi[0]) : T(0));
        qxa = x0 ? T(sd.qlo[0]) : (x1 ? T(sd.qhi[0]) : T(0));
        ey = y0 ? T(sd.elo[1]) : (y1 ? T(sd.ehi[1]) : T(0));
        qy = y0 ? T(sd.qlo[1]) : (y1 ? T(sd.qhi[1]) : T(0));
        zqlo = uniform(T(sd.qlo[2]));
        zqhi = uniform(T(sd.qhi[2]));
      }
      // inverse diagonal of the pair by z row kind (mid, vertex, ends); 0 on
      // nodes that do not exist, which keeps them at zero
      T dam, dav, dbm, dbv;
      // (those of the end planes wait in private memory: a block needs them once a sweep)
      const int nthreads = blockDim.x;
      P4<T>* const hrs = reinterpret_cast<P4<T>*>(a.chip_halo) + (size_t)ticket * kChipPrivate * nthreads;
      {
        T dal, dah, dbl, dbh;
        const T a1 = kxa * ry.m0 + mxa * ry.k0, a2 = mxa * ry.m0;
        const T b1 = kxb * ry.m0 + mxb * ry.k0, b2 = mxb * ry.m0;
        T qa1 = T(0), qa2 = T(0), qa3 = T(0), qb1 = T(0), qb2 = T(0), qb3 = T(0);
        if constexpr (Q) {
          const T kxp = kxa - exa, kyp = ry.k0 - ey;
          qa1 = qxa * kyp + qy * kxp;
          qa2 = qxa * ry.m0 + qy * mxa;
          qa3 = kxp * ry.m0 + mxa * kyp;
          qb1 = qy * kxb;
          qb2 = qy * mxb;
          qb3 = kxb * ry.m0 + mxb * kyp;
        }
        // kp: the row's centre without the Robin coefficient
        auto inv_a = [&](T k0, T kp, T m0, T q) {
          return la ? T(1) / (a1 * m0 + a2 * k0 + qa1 * m0 + qa2 * kp + q * qa3) : T(0);
        };
        auto inv_b = [&](T k0, T kp, T m0, T q) {
          return lb ? T(1) / (b1 * m0 + b2 * k0 + qb1 * m0 + qb2 * kp + q * qb3) : T(0);
        };
        dam = inv_a(kzm, kzm, mzm, T(0));
        dav = inv_a(kzv, kzv, mzv, T(0));
        dal = inv_a(kzl, T(7) * zks, mze, zqlo);
        dah = inv_a(kzh, T(7) * zks, mze, zqhi);
        dbm = inv_b(kzm, kzm, mzm, T(0));
        dbv = inv_b(kzv, kzv, mzv, T(0));
        dbl = inv_b(kzl, T(7) * zks, mze, zqlo);
        dbh = inv_b(kzh, T(7) * zks, mze, zqhi);
        hrs[4 * nthreads + tid] = P4<T>{dal, dbl, dah, dbh};
      }
      // ------------------------------------------------ halo planes
      // a mid-point plane couples only to the planes next to it
      const bool mid0 = ((zb0 + zk) & 1) != 0, mid1 = ((zb1 - 1 + zk) & 1) != 0;
      const int nlo = tau > 0 ? (mid0 ? 1 : 2) : 0, nhi = tau < TM - 1 ? (mid1 ? 1 : 2) : 0;
      // (r and s of the lower two and the upper two in private memory, hrs[0 .. 4))
      const int cs = a.chip_slots;
      // w of the edge planes: [member][lower, upper][parity][plane][slot]
      constexpr int MW = mail_words<T>;
      unsigned long long* const mail =
          reinterpret_cast<unsigned long long*>(a.chip_mail) + (size_t)team * TM * 8 * cs * MW;
      P2<T>* const wg = reinterpret_cast<P2<T>*>(a.chip_w) + (size_t)ticket * (P + kChipAhead) * nthreads;
      // ------------------------------------------------ state of the solve
      const T tsig = T(ldexp(1.0, sexp));
      T ra[P], rb[P], sa[XG ? 1 : P], sb[XG ? 1 : P];
      {
        const T* __restrict__ r0 = reinterpret_cast<const T*>(a.r) + off;
        const int ca = ia + nx * row;
        auto r_at = [&](int k, T& va, T& vb) {
          va = la ? at(r0, uint32_t(ca + S * k)) * tsig : T(0);
          vb = lb ? at(r0, uint32_t(ca + 1 + S * k)) * tsig : T(0);
        };
        unroll<0, P>([&](auto ic) {
          constexpr int i = decltype(ic)::value;
          ra[i] = rb[i] = T(0);
          if constexpr (!XG) sa[i] = sb[i] = T(0);
          if (i < zlen) r_at(zb0 + i, ra[i], rb[i]);
        });
        T z = T(0);  // (opaque: not to be kept in registers from one subdomain to the next)
        asm volatile("" : "+v"(z));
        for (int i = 0; i < zlen; ++i) {
          if (live) {
            px[i * nslots + slot] = P4<T>{z, z, z, z};
            if constexpr (WL) wl[i * nslots + slot] = P2<T>{z, z};
          }
          if constexpr (!WL) wg[i * nthreads + tid] = P2<T>{z, z};
          if constexpr (XG) xg[i * nthreads + tid] = P2<T>{z, z};
        }
        for (int h = 0; h < 4; ++h) {
          if (h < 2 ? h >= nlo : h - 2 >= nhi) continue;
          T va, vb;
          r_at(h < 2 ? zb0 - nlo + h : zb1 + h - 2, va, vb);
          hrs[h * nthreads + tid] = P4<T>{va, vb, z, z};
        }
        for (int i0 = 0; i0 < 2 * opn; i0 += nthreads)  // (uniform trips, see lds_zero)
          if (i0 + tid < 2 * opn) opl[i0 + tid] = P2<T>{z, z};
      }
      __syncthreads();
      // LDS addresses: two rows below this pair's place in the first operand
      // plane (rows are at constant offsets from there), w, and p and x
      const uint32_t rowb = (uint32_t)np * (uint32_t)sizeof(P2<T>), opb = (uint32_t)opn * (uint32_t)sizeof(P2<T>);
      const uint32_t op0 = lds_address(opl) + (uint32_t)slot * (uint32_t)sizeof(P2<T>);
      const uint32_t lds0 = lds_address(smem), px0 = lds_address(px) - 2 * lds0;
      const uint32_t plane = (uint32_t)nslots * (uint32_t)sizeof(P2<T>);
      // ------------------------------------------------ CG iterations
      // Sweep 0 runs with alpha = beta = 0 on w = s = p = x = 0: it leaves r,
      // p = D^-1 r and w = A D^-1 r, from which the first step follows.
      T alpha = T(0), beta = T(0), last_alpha = T(0);
      double gamma = 0.0, dalpha = 0.0;
      P4<T> hv[2];  // r, s of a side's halo planes (an unused one repeats)
      hv[0] = hv[1] = P4<T>{T(0), T(0), T(0), T(0)};
      P2<T> wlo[2], whi[2];  // w of the halo planes (none before the first sweep)
      wlo[0] = wlo[1] = whi[0] = whi[1] = P2<T>{T(0), T(0)};
      for (int n = 0;; ++n, ++seq) {
        T ag = T(0), ad = T(0), ar = T(0);
        T a0a = T(0), a0b = T(0), a1a = T(0), a1b = T(0), a2a = T(0), a2b = T(0), a3a = T(0), a3b = T(0);
        T ca = T(0), cb = T(0), u1a = T(0), u1b = T(0), u2a = T(0), u2b = T(0);
        const int wr = (int)(seq & 1u);
        // Running offsets and the closure index of the plane in the pass, made
        // opaque: otherwise every unrolled plane's addresses and row
        // coefficients are hoisted out of the sweep and spilled.
        uint32_t ob = op0, q = lds0 + (uint32_t)slot * (uint32_t)sizeof(P2<T>), g = (uint32_t)tid * (uint32_t)sizeof(P2<T>);
        int c = zb0 - nlo + zk, left = zlen;
        asm volatile("" : "+v"(ob), "+v"(q), "+v"(g), "+v"(c), "+v"(left));
        c = uniform(c);
        left = uniform(left);
        uint32_t gs = g;  // w's store offset (private buffer)
        // x takes the steps of this sweep and the last one, on even sweeps
        const bool xturn = XG && (n & 1) == 0 && n > 0;
        P2<T> xv[XG ? kChipAhead : 1];
        if constexpr (XG) {
#pragma unroll
          for (int j = 0; j < kChipAhead; ++j) {
            xv[j] = P2<T>{T(0), T(0)};
            if (xturn) xv[j] = *reinterpret_cast<const P2<T>*>(reinterpret_cast<const char*>(xg + j * nthreads) + g);
          }
        }
        uint32_t oflip = ob * 2 + opb;  // ob + the other plane's offset
        P4<T> pxv = lds_at<P4<T>>(px0 + 2 * q);
        P2<T> wv[kChipAhead];
        if constexpr (WL) {
          wv[0] = lds_at<P2<T>>(q);
        } else {
#pragma unroll
          for (int j = 0; j < kChipAhead; ++j)
            wv[j] = *reinterpret_cast<const P2<T>*>(reinterpret_cast<const char*>(wg + j * nthreads) + g);
        }
        // inverse diagonal at closure index k (uniform)
        auto dinv = [&](int k, T& va, T& vb) {
          const bool m = (k & 1) != 0;
          va = pick(m, dam, dav);
          vb = pick(m, dbm, dbv);
          if (k == 0 || k == zne2) {
            asm volatile("");  // a branch: only the subdomain's end planes come here
            const P2<T> v = reinterpret_cast<const P2<T>*>(hrs + 4 * nthreads + tid)[k == 0 ? 0 : 1];
            va = v.a;
            vb = v.b;
            asm volatile("" : "+v"(va), "+v"(vb));  // waits for the load here, not on every plane
          }
        };
        // operand D^-1 r of own plane i (closure index k), all CG updates of
        // the plane, the operand into the LDS plane at o
        auto make_own = [&](auto ic, int k, T& ua, T& ub, uint32_t o) {
          constexpr int i = decltype(ic)::value;
          T da, db;
          dinv(k, da, db);
          const P2<T> w = wv[WL ? 0 : i % kChipAhead];
          const T p0a = pxv.a, p0b = pxv.b;
          T pa = fma(beta, p0a, da * ra[i]), pb = fma(beta, p0b, db * rb[i]);
          // second half of the record: x, or s
          T ea, eb;
          T& sai = XG ? ea : sa[XG ? 0 : i];
          T& sbi = XG ? eb : sb[XG ? 0 : i];
          if constexpr (XG) {
            ea = pxv.c;
            eb = pxv.d;
          } else {
            ea = fma(alpha, pa, pxv.c);
            eb = fma(alpha, pb, pxv.d);
          }
          // (the old record is used up before the next one's load, which then
          // takes its registers)
          asm volatile("" : "+v"(ea), "+v"(eb));
          if constexpr (!XG) asm volatile("" : "+v"(pa), "+v"(pb));
          const uint32_t pq = px0 + 2 * q;
          q += plane;
          asm("" : "+v"(q));
          if constexpr (i + 1 < P) {
            // (an idle lane reads slot 0: it stores nothing, its inverse
            // diagonal is 0 and its sums are dropped at the end of the sweep)
            pxv = lds_at<P4<T>>(px0 + 2 * q);
            if constexpr (WL) wv[0] = lds_at<P2<T>>(q);
          }
          if constexpr (XG) {
            if (xturn) {
              P2<T>& x = xv[i % kChipAhead];
              *reinterpret_cast<P2<T>*>(reinterpret_cast<char*>(xg) + g) =
                  P2<T>{fma(alpha, pa, fma(last_alpha, p0a, x.a)), fma(alpha, pb, fma(last_alpha, p0b, x.b))};
              if constexpr (i + 1 < P)
                x = *reinterpret_cast<const P2<T>*>(reinterpret_cast<const char*>(xg + kChipAhead * nthreads) + g);
            }
          }
          if constexpr ((!WL || XG) && i + 1 < P) {
            if constexpr (!WL)
              wv[i % kChipAhead] =
                  *reinterpret_cast<const P2<T>*>(reinterpret_cast<const char*>(wg + kChipAhead * nthreads) + g);
            g += (uint32_t)nthreads * (uint32_t)sizeof(P2<T>);
            asm("" : "+v"(g));
          }
          sai = w.a + beta * sai;
          sbi = w.b + beta * sbi;
          ra[i] -= alpha * sai;
          rb[i] -= alpha * sbi;
          ua = da * ra[i];
          ub = db * rb[i];
          ag += ra[i] * ua;
          ag += rb[i] * ub;
          ar += ra[i] * ra[i];
          ar += rb[i] * rb[i];
          if (live) {
            lds_at<P4<T>>(pq) = P4<T>{pa, pb, ea, eb};
            lds_at<P2<T>>(o + 2 * rowb) = P2<T>{ua, ub};
          }
        };
        // the same for halo plane h (r and s only)
        auto make_halo = [&](int h, int k, P4<T> v, P2<T> w, T& ua, T& ub, uint32_t o) {
          T da, db;
          dinv(k, da, db);
          v.c = w.a + beta * v.c;
          v.d = w.b + beta * v.d;
          v.a -= alpha * v.c;
          v.b -= alpha * v.d;
          hrs[h * nthreads + tid] = v;
          ua = da * v.a;
          ub = db * v.b;
          if (live) lds_at<P2<T>>(o + 2 * rowb) = P2<T>{ua, ub};
        };
        auto load_halo = [&](int side, int count) {
#pragma unroll
          for (int h = 0; h < 2; ++h) hv[h] = hrs[(2 * side + min(h, count - 1)) * nthreads + tid];
        };
        // waits for this sweep's w on the halo planes (a neighbour's edge: the
        // lower side's planes are the last of the lower member's upper edge);
        // true if it did not come in time
        auto fetch_mail = [&]() {
          if (!live || (nlo | nhi) == 0) return false;
          if (nlo) load_halo(0, nlo);  // (for the next sweep)
          const unsigned long long* lo = mail + (size_t)(((tau - 1) * 8 + 4 + 2 * wr + 2 - nlo) * cs + slot) * MW;
          const unsigned long long* hi = mail + (size_t)(((tau + 1) * 8 + 2 * wr) * cs + slot) * MW;
          const size_t up = (size_t)cs * MW;
          const unsigned want = seq + ((unsigned)a.tag_skew << 31);
          const unsigned long long t0 = wall_clock64();
          for (;;) {
            bool ok = true;
            if (nlo) ok = mail_read(lo, want, wlo[0]);
            if (nlo == 2) ok = mail_read(lo + up, want, wlo[1]) && ok;
            if (nhi) ok = mail_read(hi, want, whi[0]) && ok;
            if (nhi == 2) ok = mail_read(hi + up, want, whi[1]) && ok;
            if (ok) return false;
            if (wall_clock64() - t0 > ticks) return true;
          }
        };
        // one operand plane (closure index k, own operand ua, ub): y- and
        // x-pass, the scatter along z; out: A u two planes below
        struct Y {
          P2<T> m1, p1, m2, p2;
        };
        auto read_rows = [&](uint32_t o) {
          return Y{lds_at<P2<T>>(o + rowb), lds_at<P2<T>>(o + 3 * rowb), lds_at<P2<T>>(o), lds_at<P2<T>>(o + 4 * rowb)};
        };
        auto pass = [&](int k, const Y& y, T ua, T ub, T& oa, T& obv) {
          const T s1a = y.m1.a + y.p1.a, s1b = y.m1.b + y.p1.b, s2a = y.m2.a + y.p2.a, s2b = y.m2.b + y.p2.b;
          const T fa = my0 * ua + my1 * s1a + my2 * s2a, fb = my0 * ub + my1 * s1b + my2 * s2b;
          const T va = ky0 * ua + ky1 * s1a + ky2 * s2a, vb = ky0 * ub + ky1 * s1b + ky2 * s2b;
          const T fl = from_below(fa), fm = from_below(fb), fr = from_above(fa);
          const T vl = from_below(va), vm = from_below(vb), vr = from_above(va);
          const T f1a = fm + fb, f2a = fl + fr, f1b = fa + fr;
          const T v1a = vm + vb, v2a = vl + vr, v1b = va + vr;
          T Sa = kxa * fa + kx1 * f1a + ksx * f2a + mxa * va + mx1 * v1a - msx * v2a;
          T Ta = mxa * fa + mx1 * f1a - msx * f2a;
          T Sb = kxb * fb + kx1 * f1b + mxb * vb + mx1 * v1b;
          T Tb = mxb * fb + mx1 * f1b;
          T za = T(0), zb = T(0);
          if constexpr (Q) {
            // second-order faces (see zmarch); the operand's x-neighbours
            // come from the adjacent lanes too (an idle lane's operand is 0)
            const T pl = from_below(ua), pm = from_below(ub), pr = from_above(ua);
            const T p1a = pm + ub, p2a = pl + pr, p1b = ua + pr;
            const T pma = mxa * ua + mx1 * p1a - msx * p2a, pmb = mxb * ub + mx1 * p1b;
            const T pka = (kxa - exa) * ua + kx1 * p1a + ksx * p2a, pkb = kxb * ub + kx1 * p1b;
            const T sfa = qxa * (va - ey * ua) + qy * pka, sfb = qy * pkb;
            const T tfa = qxa * fa + qy * pma, tfb = qy * pmb;
            if (k == 0 || k == zne2) {
              const T zq = pick(k == 0, zqlo, zqhi), ez = pick(k == 0, zelo, zehi);
              za = zq * (Sa - exa * fa - ey * pma) - ez * tfa;
              zb = zq * (Sb - ey * pmb) - ez * tfb;
            }
            Sa += sfa;
            Sb += sfb;
            Ta += tfa;
            Tb += tfb;
          }
          const T c1a = mz1 * Sa + kz1 * Ta, c1b = mz1 * Sb + kz1 * Tb;
          if ((k & 1) != 0) {
            asm volatile("");  // a branch: a mid-point plane reaches only the planes next to it
            oa = a0a;
            obv = a0b;
            a0a = a1a + c1a;
            a0b = a1b + c1b;
            a1a = a2a + (mzm * Sa + kzm * Ta);
            a1b = a2b + (mzm * Sb + kzm * Tb);
            a2a = a3a + c1a;
            a2b = a3b + c1b;
            a3a = a3b = T(0);
          } else {
            T zk0 = kzv, zm0 = mzv;
            if (k == 0 || k == zne2) {
              asm volatile("");  // a branch, see dinv
              zk0 = pick(k == 0, kzl, kzh);
              zm0 = mze;
            }
            const T c2a = zks * Ta - zms * Sa, c2b = zks * Tb - zms * Sb;
            oa = a0a + c2a;
            obv = a0b + c2b;
            a0a = a1a + c1a;
            a0b = a1b + c1b;
            a1a = a2a + (zm0 * Sa + zk0 * Ta);
            a1b = a2b + (zm0 * Sb + zk0 * Tb);
            if constexpr (Q) {
              a1a += za;
              a1b += zb;
            }
            a2a = a3a + c1a;
            a2b = a3b + c1b;
            a3a = c2a;
            a3b = c2b;
          }
        };
        // w of an own plane is complete: back = planes from it to the next own
        // plane to make (the running offsets' place)
        auto store = [&](int back, T oa, T obv) {
          const T wa = la ? oa : T(0), wb = lb ? obv : T(0);
          ad += wa * u2a;
          ad += wb * u2b;
          if constexpr (WL) {
            if (live) lds_at<P2<T>>(q - (uint32_t)back * plane) = P2<T>{wa, wb};
          } else {
            *reinterpret_cast<P2<T>*>(reinterpret_cast<char*>(wg) + gs) = P2<T>{wa, wb};
            gs += (uint32_t)nthreads * (uint32_t)sizeof(P2<T>);
            asm("" : "+v"(gs));
          }
        };
        auto carry = [&](T na, T nb) {
          u2a = u1a;
          u2b = u1b;
          u1a = ca;
          u1b = cb;
          ca = na;
          cb = nb;
          ob = oflip - ob;
          asm("" : "+v"(ob));
          c = scalar_add<1>(c);
        };
        T na = T(0), nb = T(0), oa, obv;
        if (nlo) {
          if (n == 0) load_halo(0, nlo);
          make_halo(0, c, hv[0], wlo[0], ca, cb, ob);
          if (nlo == 2) {
            __syncthreads();
            const Y y = read_rows(ob);
            make_halo(1, c + 1, hv[1], wlo[1], na, nb, oflip - ob);
            pass(c, y, ca, cb, oa, obv);
            carry(na, nb);
          }
          __syncthreads();
          const Y y = read_rows(ob);
          make_own(std::integral_constant<int, 0>(), c + 1, na, nb, oflip - ob);
          pass(c, y, ca, cb, oa, obv);
          carry(na, nb);
        } else {
          make_own(std::integral_constant<int, 0>(), c, ca, cb, ob);
        }
        // left: own planes whose pass is to come (a running count, so that the
        // tests of the unrolled planes are not all kept in registers)
        unroll<0, P>([&](auto ic) {
          constexpr int i = decltype(ic)::value;
          if (left > 0) {
            __syncthreads();
            const Y y = read_rows(ob);
            const bool more = i + 1 < P && left > 1;
            if constexpr (i + 1 < P) {
              if (more) make_own(std::integral_constant<int, i + 1>(), c + 1, na, nb, oflip - ob);
            }
            const bool last = !more && nhi;
            if (last) load_halo(1, nhi);
            pass(c, y, ca, cb, oa, obv);
            if (last) make_halo(2, c + 1, hv[0], whi[0], na, nb, oflip - ob);
            if constexpr (i >= 2) store(more ? 4 : 3, oa, obv);
            carry(na, nb);
            left = scalar_add<-1>(left);
          }
        });
        if (nhi) {
          __syncthreads();
          const Y y = read_rows(ob);
          if (nhi == 2) make_halo(3, c + 1, hv[1], whi[1], na, nb, oflip - ob);
          pass(c, y, ca, cb, oa, obv);
          if (zlen >= 2) store(2, oa, obv);
          carry(na, nb);
          if (nhi == 2) {
            __syncthreads();
            const Y y2 = read_rows(ob);
            pass(c, y2, ca, cb, oa, obv);
            store(1, oa, obv);
            carry(na, nb);
          }
        }
        // the planes whose last neighbours do not exist
        for (int i = zlen + nhi - 2; i < zlen; ++i) {
          oa = a0a;
          obv = a0b;
          a0a = a1a;
          a0b = a1b;
          if (i >= 0) store(zlen - i, oa, obv);
          carry(T(0), T(0));
        }
        // the edge planes go out last: written within the sweep, every later
        // load of the sweep would wait for these stores to reach memory
        if (TM > 1 && live) {
          const uint32_t w0 = lds0 + (uint32_t)slot * (uint32_t)sizeof(P2<T>);
          unsigned long long* const m = mail + (size_t)((tau * 8 + 2 * wr) * cs + slot) * MW;
#pragma unroll
          for (int e4 = 0; e4 < 4; ++e4) {
            if (e4 < 2 ? tau == 0 : tau == TM - 1) continue;
            const int i = e4 < 2 ? e4 : zlen - 4 + e4;
            P2<T> v;
            if constexpr (WL) v = lds_at<P2<T>>(w0 + (uint32_t)i * plane);
            else v = wg[i * nthreads + tid];
            mail_write(m + (size_t)((e4 < 2 ? e4 : e4 + 2) * cs) * MW, seq, v.a, v.b);
          }
        }
        double g0 = double(ag), d0 = double(ad);
        if constexpr (sizeof(T) < sizeof(double)) {
          // every step length and direction of the solve descends from the first
          // gamma and delta: FP64 products and sums, as in k_fused_cg (the sums of the
          // later sweeps are the inner precision's within a thread there too), from
          // the stored p, which is D^-1 r still (forming it again: more code to fetch,
          // 37 x 29 x 23 elements in 27 17.23 ms a solve, 16.99 so, 16.93 without these
          // sums). Unlikely, so that the code lies outside the sweeps' (amid them 128^3
          // in 512, second order, 1004 to 1009 ms, there 996 to 999, without 991).
          if (__builtin_expect(n == 0, 0)) {
            g0 = d0 = 0.0;
            uint32_t qw = lds0 + (uint32_t)slot * (uint32_t)sizeof(P2<T>), gw = (uint32_t)tid * (uint32_t)sizeof(P2<T>);
            int more = zlen;
            asm volatile("" : "+v"(qw), "+v"(gw), "+v"(more));
            more = uniform(more);
            unroll<0, P>([&](auto ic) {
              constexpr int i = decltype(ic)::value;
              if (more > 0) {
                const P2<T> u = lds_at<P2<T>>(px0 + 2 * qw);
                P2<T> w;
                if constexpr (WL) w = lds_at<P2<T>>(qw);
                else w = *reinterpret_cast<const P2<T>*>(reinterpret_cast<const char*>(wg) + gw);
                g0 += double(ra[i]) * double(u.a);
                g0 += double(rb[i]) * double(u.b);
                d0 += double(w.a) * double(u.a);
                d0 += double(w.b) * double(u.b);
                qw += plane;
                if constexpr (!WL) gw += (uint32_t)nthreads * (uint32_t)sizeof(P2<T>);
                asm("" : "+v"(qw), "+v"(gw));
                more = scalar_add<-1>(more);
              }
            });
          }
        }
        if (!live) g0 = d0 = 0.0, ar = T(0);
        double acc[3] = {g0, d0, double(ar)};
        chip_sum(acc, sh, a, s, tau, TM, epoch++, ticks, tfail, fetch_mail);
        ticks = a.spin_ticks;
        if (tfail) {
          brk |= kBrkBarrier;
          break;
        }
        if (!isfinite(acc[0]) || !isfinite(acc[1]) || !isfinite(acc[2])) {
          t = n;
          brk |= kBrkNonFinite;
          break;
        }
        t = n;
        if (n == 0) {
          if (!(acc[1] > 0.0)) {
            brk |= kBrkCurvature;
            break;
          }
          gamma = uniform(acc[0]);
          dalpha = uniform(acc[0] / acc[1]);
          alpha = uniform(T(dalpha));
          continue;
        }
        if (!(acc[2] > stop2s) || t >= a.max_inner) {
          if ((n & 1) != 0) xstep = alpha;
          break;
        }
        last_alpha = alpha;
        const double dbeta = acc[0] / gamma;
        const double den = acc[1] - dbeta * acc[0] / dalpha;
        if (!(den > 0.0)) {
          brk |= isfinite(den) ? kBrkCurvature : kBrkNonFinite;
          break;
        }
        dalpha = uniform(acc[0] / den);
        gamma = uniform(acc[0]);
        alpha = uniform(T(dalpha));
        beta = uniform(T(dbeta));
      }
      seq = mail_next_job(seq);  // (not for a subdomain without a sweep)
    }
    // the next subdomain of this team: the first member takes it and leaves it
    // in a spare word of this subdomain's slots for the others
    if (tid == 0 && tau == 0) {
      sh.job = atomicAdd(&a.queue[1], 1) + a.n_teams;
      if (TM > 1) {
        unsigned long long* w = reinterpret_cast<unsigned long long*>(
            chip_part(a, s) + kTeamSlot - 1);
        st_coh(w, (unsigned long long)sh.job + 1ull);
      }
    }
    // a subdomain whose solve broke down keeps its iterate (the host reports it)
    if (t > 0 && !brk) {
      const double isig = ldexp(1.0, -sexp);
      double* __restrict__ ub = a.u + off;
      const int c0 = ia + nx * row + S * zb0;
      if (live) {
#pragma unroll 4
        for (int i = 0; i < zlen; ++i) {
          const P4<T> v = px[i * nslots + slot];
          P2<T> x{v.c, v.d};
          if constexpr (XG) {
            x = xg[i * (int)blockDim.x + tid];
            x = P2<T>{fma(xstep, v.a, x.a), fma(xstep, v.b, x.b)};
          }
          if (la) at(ub, uint32_t(c0 + S * i)) += double(x.a) * isig;
          if (lb) at(ub, uint32_t(c0 + 1 + S * i)) += double(x.b) * isig;
        }
      }
    }
    if (tid == 0 && brk) atomicOr(a.flags, brk);
    if (tid == 0 && tau == 0) {
      a.scal[s].iters = t;
      a.scal[s].breakdown = brk;
      a.scal[s].done = 1;
      atomicAdd(&a.iters_total[0], (unsigned long long)t);
      atomicAdd(&a.iters_total[1], fused_bytes(sd, t, sizeof(T)));
    }
    if (tid == 0 && tau != 0) {
      const unsigned long long* w = reinterpret_cast<const unsigned long long*>(
          chip_part(a, s) + kTeamSlot - 1);
      const unsigned long long t0 = wall_clock64();
      unsigned long long v = ld_coh(w);
      while (v == 0ull && wall_clock64() - t0 <= ticks) v = ld_coh(w);
      sh.job = v ? (int)(v - 1ull) : -1;
    }
    __syncthreads();
    job = uniform(sh.job);
    // a member that gave up leaves the team (so do the others, at their own
    // bounded waits); nothing more can be solved with it
    if (brk & kBrkBarrier) return;
    if (job < 0) {
      if (tid == 0) atomicOr(a.flags, (int32_t)kBrkBarrier);
      return;
    }
    __syncthreads();
  }
}

}  // namespace sos
