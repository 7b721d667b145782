// gfx950 kernel of the tracklet fit and track following (Rohr, LHCP 2017,
// Sec. 2 and Fig. 1c), one tracklet per lane: seed on the chain's first hit
// with the direction of its end points; pass 1 updates with the chain and
// follows outward picking the nearest window hit with chi2 <= pick_chi2 (stop
// after max_miss empty rows); pass 2 restarts at the outermost hit with the
// pass-1 covariance x refit_inflate, refits inward through all pass-1 hits
// and continues below the chain start.
//
// The state's z is kept relative to zr, the z of the chain's first hit:
// measurements enter as z_hit - zr (exact for a track's own hits) and the
// outputs add zr back.  Time frames place z' tens of metres from the
// sector's origin (Sec. 5), where an absolute FP32 z would carry rounding
// errors comparable with the fit's resolution.
//
// The kernel has two forms with the same operation sequence per tracklet and
// takes one by the number of tracklets it finds:
//   few   each lane runs its tracklet's loops one after the other, spread over
//         as many waves as there are, up to two per SIMD.  The time is that of
//         the longest tracklet's steps, and a lone wave issues an instruction
//         every four to seven cycles, so a wave of one tracklet has loops that
//         hold nothing but their own phase, and one of several a loop per pass.
//   many  a persistent per-lane state machine: every iteration performs one
//         row step of whatever phase the lane is in, and a lane whose
//         tracklet is done takes the next one of its wave's pool, so that
//         lanes stay busy while tracklets of very different lengths share a
//         wave.
#include <hip/hip_runtime.h>

#include "tpcca_internal.h"
#include "tpcca_kernels.h"
#include "tpcca_dev.h"
#include "tpcca_kf.h"
#include "tpcca_fit.h"

#include <algorithm>
#include <map>
#include <mutex>

namespace tpcca {

// ----------------------------------------------------------------- work ---
// Slice x of n items cut into nsl.
__device__ __forceinline__ void pool_slice(int n, int nsl, int x, int &lo, int &hi) {
  const int q = n / nsl, r = n - q * nsl;
  lo = q * x + min(x, r);
  hi = q * (x + 1) + min(x + 1, r);
}

// Few tracklets: the waves that share them, and the most they take.
constexpr int kFewWaves = 2048;
constexpr int kFewMax = 64 * kFewWaves;

// The wave's share [lo, hi) of a few tracklets: contiguous slices of the order
// per XCD (block b runs on XCD b mod 8), cut evenly over its waves, the first
// waves of all blocks before the second ones: the dispatcher fills CU after
// CU with blocks, and waves that share a CU slow each other's instruction
// fetch (a sector's 77 tracklets: fit 0.47 ms one to a CU, 0.63 two, 0.85
// four).
__device__ __forceinline__ void few_share(int n, int &lo, int &hi) {
  const int wpb = (int)blockDim.x >> 6, wid = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int nb = (int)gridDim.x, b = (int)blockIdx.x;
  const int nsl = min(kXcds, nb), x = b % kXcds, nbx = (nb - x + kXcds - 1) / kXcds;
  const int nwx = min(nbx * wpb, kFewWaves / kXcds), j = wid * nbx + b / kXcds;
  int s0, s1;
  pool_slice(n, nsl, x, s0, s1);
  const int per = (s1 - s0 + nwx - 1) / nwx;
  lo = min(s1, s0 + j * per);
  hi = j < nwx ? min(s1, lo + per) : lo;
}

// A wave's share of many tracklets: a first share per wave, then shares
// claimed from a work counter.  Up to kEqualShare per wave the first share is all
// there is: claims of 64 after the first 64 then go to some waves only.  Whole
// passes on 4096 waves, claims against equal shares, of a batch or frame alone
// and per batch of two in flight (us):
//    67 to a wave (frame of 40 events)   2950 / 2970   2890 / 2850
//   107 (64 minimum-bias events)         4885 / 4570   4625 / 4690
//   113 (frame of 48 events)             4845 / 4495   4630 / 4625
//   125 (80 minimum-bias events)         5605 / 5325   5470 / 5450
//   135 (frame of 56 events)             5785 / 5340   5500 / 5550
//   167 (64 events)                      6870 / 6345   6800 / 6795
//   203 (80 events)                      8210 / 7685   8355 / 8360
//   278 (128 events)                    10900 / 10275 11695 / 11660
// Alone, evenness wins up to some 170; with two in flight the other batch fills
// the uneven end, and claims win from some 100 on.  The line lies between.
// Claims of at most half of what is left per wave, instead of four times that:
// 128 events alone 10.90 -> 10.75 ms, two in flight 10.08 -> 10.19 per frame.
constexpr int kEqualShare = 128;
struct Pool {
  int next = 0, end = 0;  // claimed, not yet started
  int part = 0, tried = 0;
  int seen = 0;           // the work counter as of this wave's last claim
  int base = 0;           // order positions handed out without the counter
  bool exhausted = false;
};

__device__ __forceinline__ Pool pool_start(const ParamsDev &P, int n) {
  Pool p;
  const int wpb = (int)blockDim.x >> 6, wid = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int nw = (int)gridDim.x * wpb;
  if (P.kf_xcd) {
    p.part = (int)blockIdx.x % kXcds;
  } else {
    const int per = (n + nw - 1) / nw;
    const int first = max(64, per <= kEqualShare ? per : min(P.kf_pool, 4 * per));
    p.next = min(n, ((int)blockIdx.x * wpb + wid) * first);
    p.end = min(n, p.next + first);
    p.base = p.seen = nw * first;
  }
  return p;
}

// Claims the next tracklets of the wave's slice with one atomic per wave:
// kf_pool neighbouring ones while many remain; in the last stretch (less than
// a quarter pool per wave left, judged from this wave's previous claim) fewer,
// but never fewer than the idle lanes, so that at the end no wave holds a
// private backlog.  With slices per XCD (kf_xcd), the waves of an XCD drain
// its slice first and then help with the following ones.
__device__ __forceinline__ void pool_claim(const ParamsDev &P, Pool &p, int32_t *counter, int n, int n_idle,
                                           int lane) {
  const int nsl = P.kf_xcd ? kXcds : 1;
  int lo = 0, hi = n;
  if (nsl > 1) pool_slice(n, nsl, p.part, lo, hi);
  const int nw = (int)((gridDim.x * blockDim.x) >> 6);
  const int want = max(n_idle, min(P.kf_pool, 4 * (((hi - lo) - p.seen) / nw)));
  int got = 0;
  if (p.base < hi - lo) {
    if (lane == 0) got = atomicAdd(&counter[p.part], want);
    got = __shfl(got, 0, 64);
  }
  got += p.base;
  p.seen = got + want;
  if (got < hi - lo) {
    p.next = lo + got;
    p.end = min(p.next + want, hi);
  } else if (++p.tried == nsl) {
    p.exhausted = true;
  } else {
    p.part = (p.part + 1) % nsl;
    p.seen = 0;
  }
}

// 16 B at p: a row's grid description, or a sorted hit (8 B) and the next.
__device__ __forceinline__ int4 load16(const void *p) {
  int4 v;
  __builtin_memcpy(&v, __builtin_assume_aligned(p, 8), 16);
  return v;
}

// Nearest hit (dy^2 + dz^2, ties to the lower ID) of the row described by t
// inside the prediction window; -1 if none; its coordinates are returned
// in bc.
// The state's z is relative to zr; the bins are looked up around the absolute
// prediction zr + z with a margin that covers its rounding.
template <int kQ>
__device__ __forceinline__ int kf_search(const Bufs &B, const ParamsDev &P, const RowTab &t,
                                         const KState &s, float zr, unsigned int &cands, float2 &bc) {
  // with cluster variances the roots' arguments are in kf_sqrt's range (what a
  // covariance slightly below zero leaves of a variance is 2^-24 of it or more)
  const bool mid = P.ery >= 0x1p-70f && P.erz >= 0x1p-70f;
  const float vy = s.C[0] + P.ery, vz = s.C[2] + P.erz;
  float wy = P.nsig * (mid ? kf_sqrt(vy) : sqrtf(vy));
  float wz = P.nsig * (mid ? kf_sqrt(vz) : sqrtf(vz));
  if (wy > P.wmax) wy = P.wmax;
  if (wz > P.wmax) wz = P.wmax;
  int b, e;
  bin_range(t, B.binbeg, zr + s.p[1], wz, b, e);
  cands += (unsigned int)(e - b);
  int best = -1;
  float bd2 = __builtin_inff();
  bool tie = false;
  // candidates in ascending sorted index, kQ at a time in 16-B loads of two
  // (independent loads in flight, the last ones repeated past the end); a
  // second hit at exactly the best distance (rare) is only noted.  The state
  // machine waits less with eight (a frame of 33 M clusters: 8.4 ms, 8.9 with
  // four, 9.4 with sixteen); a lone wave's loops do not.
  for (int i0 = b; i0 < e; i0 += kQ) {
    int4 c[kQ / 2];
#pragma unroll
    for (int q = 0; q < kQ / 2; ++q) c[q] = load16(B.yz + min(i0 + 2 * q, e - 1));
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
      const float cy = __int_as_float(q & 1 ? c[q / 2].z : c[q / 2].x);
      const float cz = __int_as_float(q & 1 ? c[q / 2].w : c[q / 2].y);
      const float dy = cy - s.p[0];
      const float dz = (cz - zr) - s.p[1];
      const float d2 = __builtin_fmaf(dy, dy, dz * dz);
      const bool in = (i0 + q < e) & (fabsf(dy) <= wy) & (fabsf(dz) <= wz);
      const bool lt = in & (d2 < bd2);
      tie = !lt & (tie | (in & (d2 == bd2)));
      bd2 = lt ? d2 : bd2;
      best = lt ? i0 + q : best;
      bc.x = lt ? cy : bc.x;
      bc.y = lt ? cz : bc.y;
    }
  }
  if (tie && best >= 0) {  // equal distances are decided by the lower cluster ID
    for (int i = best + 1; i < e; ++i) {
      const float2 c = B.yz[i];
      const float dy = c.x - s.p[0];
      const float dz = (c.y - zr) - s.p[1];
      if (!(fabsf(dy) <= wy && fabsf(dz) <= wz)) continue;
      if (__builtin_fmaf(dy, dy, dz * dz) == bd2 && B.sid[i] < B.sid[best]) {
        best = i;
        bc = c;
      }
    }
  }
  return best;
}

// The hit slots of a lane's tracklet move eight at a time (one aligned 32-B
// group): a lane collects a group in LDS and writes it when complete or when
// its phase ends.  Scattered stores narrower than a memory segment cost a
// read-modify-write each, so fewer, wider ones matter.  The refit reads them
// back four at a time, each four into the half they left LDS from: when pass
// 1 ends, the last four and the four before them are still there.
constexpr int kGM = kSlotGrp - 1;
static_assert(kSlotGrp == 8, "a group is two int4");

template <int kBlk>
struct Slots {
  int4 v[2][kBlk];
  __device__ __forceinline__ int32_t &at(int j) {
    return reinterpret_cast<int32_t *>(&v[(j >> 2) & 1][threadIdx.x])[j & 3];
  }
  // the group holding slot j, to the tracklet's slots
  __device__ __forceinline__ void flush(int32_t *to, int j) const {
    int4 *dst = reinterpret_cast<int4 *>(to + (j & ~kGM));
    dst[0] = v[0][threadIdx.x];
    dst[1] = v[1][threadIdx.x];
  }
};

// The state at the outermost (pass 1) or innermost (pass 2) hit, kept in LDS
// (frees registers for occupancy).
template <int kBlk>
struct Aux {
  float4 v[5][kBlk];
  float x[kBlk];
  __device__ __forceinline__ void save(const KState &st) {
    const int tid = threadIdx.x;
    v[0][tid] = make_float4(st.p[0], st.p[1], st.p[2], st.p[3]);
    v[1][tid] = make_float4(st.p[4], st.C[0], st.C[1], st.C[2]);
    v[2][tid] = make_float4(st.C[3], st.C[4], st.C[5], st.C[6]);
    v[3][tid] = make_float4(st.C[7], st.C[8], st.C[9], st.C[10]);
    v[4][tid] = make_float4(st.C[11], st.C[12], st.C[13], st.C[14]);
    x[tid] = st.x;
  }
  __device__ __forceinline__ KState load() const {
    const int tid = threadIdx.x;
    const float4 a = v[0][tid], b = v[1][tid], c = v[2][tid], d = v[3][tid], e = v[4][tid];
    return KState{{a.x, a.y, a.z, a.w, b.x},
                  {b.y, b.z, b.w, c.x, c.y, c.z, c.w, d.x, d.y, d.z, d.w, e.x, e.y, e.z, e.w},
                  x[tid]};
  }
};

// Tracklets that a wave reads ahead, and that end before it writes their claims.
// Both wait for chains of dependent reads (a start four, a claim three): one
// tracklet at a time they took 1.2 of 10.0 ms on a frame of 33 M clusters,
// where a wave's 64 lanes end one after the other.
constexpr int kSeeds = 16, kDone = 8;

// What both forms of the kernel share of a block: LDS and the work totals
// (row steps, candidates, tests, updates, iterations), which go out with one
// global atomic per counter and block, and with none from blocks without work
// (thousands of adds to the same words would serialise).
template <int kBlk>
struct FitBlock {
  Aux<kBlk> aux;
  Slots<kBlk> slot;
  int2 head[kBlk];         // the tracklet's first hit (row << 24 | cluster ID), its chain's length
  int4 seed[kBlk / 64][3][kSeeds];  // tracklets read ahead
  int2 seed_head[kBlk / 64][kSeeds];
  int4 done[kBlk / 64][kDone];      // tracklets that ended (record, hits, chi2, unit's first cluster)
  float rx[kMaxRows + 1];  // the row positions
  unsigned int steps, cands, tests, updates, iters;
};

// The set bits of a wave mask below this lane (no lane mask held in registers).
__device__ __forceinline__ int lanes_below(unsigned long long m) {
  return (int)__builtin_amdgcn_mbcnt_hi((unsigned int)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned int)m, 0u));
}

// Counts of the work done: of a lane or (all but cands in the totals) a wave.
struct Work {
  unsigned int steps = 0, cands = 0, tests = 0, updates = 0, iters = 0;
};

__device__ __forceinline__ RowTab row_bins(int4 v) {
  RowTab t;
  t.nb = v.x;
  t.bin0 = v.y;
  t.z0 = __int_as_float(v.z);
  t.inv = __int_as_float(v.w);
  return t;
}
__device__ __forceinline__ float2 hit_yz(int4 v) { return make_float2(__int_as_float(v.x), __int_as_float(v.y)); }

// A tracklet in work: its unit's row tables and first global cluster index, the
// row of the step, the chain's next hit and the one after it (sorted indices,
// -1: none), the origin of the state's z, and what the step reads of memory:
// the given hit's place or the description of the row to search.
struct Trk {
  int t, rb, ucl, r, hn, hx;
  float zr;
  int4 v;
};

// What a tracklet's start takes from memory: its unit, the chain's first hit
// (position, slot, cluster ID) and the next two, the chain's length and the
// seed's direction.
struct Seed {
  int t, u, ucl, s0, hn, hx;
  float y, z, sn, p3;
  float2 next;
  int2 head;  // cluster ID, chain length
};

// The tracklet at position pos of the processing order.
__device__ __forceinline__ Seed fit_read(const Bufs &B, const ParamsDev &P, const float *rx, int pos) {
  Seed a;
  a.t = B.kf_order[pos];
  const int g0 = B.trk_start[a.t];
  a.u = B.trk_unit[a.t];
  a.ucl = B.units[a.u].cl_begin;
  const int2 ci = B.cinfo[g0];
  a.hn = B.upc[g0];
  const int r = B.srow[g0];
  a.head = make_int2(B.sid[g0], ci.y);
  const float2 h0 = B.yz[g0], hL = B.yz[ci.x];
  a.next = B.yz[a.hn];
  a.hx = B.upc[a.hn];
  const float x0 = rx[r], xL = rx[r + ci.y - 1];
  const float dxs = xL - x0;
  const float ty = (hL.x - h0.x) / dxs;
  a.sn = ty / sqrtf(__builtin_fmaf(ty, ty, 1.0f));
  const float tz = (hL.y - h0.y) / dxs;
  a.y = h0.x;
  a.z = h0.y;
  a.p3 = tz * sqrtf(__builtin_fmaf(-a.sn, a.sn, 1.0f));
  a.s0 = slot_enc(g0, a.ucl, r);
  return a;
}

// Its fit, about to step to the chain's second hit.
template <int kBlk>
__device__ __forceinline__ void fit_start(const ParamsDev &P, FitBlock<kBlk> &S, const Seed &a, Trk &k, KState &st) {
  k.t = a.t;
  k.rb = a.u * (P.n_rows + 1);
  k.ucl = a.ucl;
  k.r = slot_row(a.s0) + 1;
  k.hn = a.hn;
  k.hx = a.hx;
  k.zr = a.z;
  k.v = make_int4(__float_as_int(a.next.x), __float_as_int(a.next.y), 0, 0);
  st.p[0] = a.y;
  st.p[1] = a.z - k.zr;
  st.p[2] = a.sn;
  st.p[3] = a.p3;
  st.p[4] = 0.0f;
#pragma unroll
  for (int q = 0; q < 15; ++q) st.C[q] = 0.0f;
  st.C[0] = P.ery;
  st.C[2] = P.erz;
  st.C[5] = P.c22;
  st.C[9] = P.c33;
  st.C[14] = P.c44;
  st.x = S.rx[k.r - 1];
  S.slot.at(0) = a.s0;
  S.head[threadIdx.x] = make_int2((int)((uint32_t)(k.r - 1) << 24) | a.head.x, a.head.y);
}

template <int kBlk>
__device__ __forceinline__ void fit_failed(const Bufs &B, const FitBlock<kBlk> &S, int t) {
  const int2 hd = S.head[threadIdx.x];
  kf_fail(B, t, hd.x & 0xFFFFFF, hd.y);
}

// The end of pass 1 (n1 hits): its last (partial) slot group goes to memory
// (the slots after n1 are written again by pass 2 or never read), its state to
// the record, and the state restarts for pass 2.
template <int kBlk>
__device__ __forceinline__ void fit_turn(const Bufs &B, const ParamsDev &P, FitBlock<kBlk> &S, const Trk &k, int n1,
                                         int32_t *slots, KState &st) {
  if (n1 & kGM) S.slot.flush(slots, n1 - 1);
  tpcca_tracklet_t &o = B.trk[k.t];
  st = S.aux.load();
  o.row_out = slot_row(S.slot.at(n1 - 1));
#pragma unroll
  for (int q = 0; q < 5; ++q) o.p_out[q] = q == 1 ? st.p[1] + k.zr : st.p[q];
#pragma unroll
  for (int q = 0; q < 15; ++q) o.cov_out[q] = st.C[q];
  o.x_out = st.x;
  kf_restart(P, st);
}

// A hit picked up below the chain start: its slot (number nh).
template <int kBlk>
__device__ __forceinline__ void fit_slot_in(FitBlock<kBlk> &S, int n1, int nh, int32_t *slots, int32_t v) {
  S.slot.at(nh) = v;
  if ((nh & ~kGM) < n1)  // a group shared with pass-1 slots: this slot alone
    slots[nh] = v;
  else if ((nh & kGM) == kGM)
    S.slot.flush(slots, nh);
}

// The end of pass 2: the record; returns whether the tracklet has enough hits.
template <int kBlk>
__device__ __forceinline__ bool fit_done(const Bufs &B, const ParamsDev &P, FitBlock<kBlk> &S, const Trk &k, int n1,
                                         int nh, float chi2, int32_t *slots) {
  tpcca_tracklet_t &o = B.trk[k.t];
  const int2 hd = S.head[threadIdx.x];
  // the last partial group of pass-2 slots (one that does not share pass-1
  // slots) goes to memory
  const int jl = nh - 1;
  if (nh > n1 && (jl & kGM) != kGM && (jl & ~kGM) >= n1) S.slot.flush(slots, jl);
  const KState a = S.aux.load();
  o.start_id = hd.x & 0xFFFFFF;
  o.n_chain = hd.y;
  o.n_hits = nh;
  o.n_pass1 = n1;
  o.ndf = 2 * nh - 5;
  o.row_ref = nh > n1 ? slot_row(S.slot.at(jl)) : slot_row(hd.x);
  o.x_ref = a.x;
  o.chi2 = chi2;
#pragma unroll
  for (int q = 0; q < 5; ++q) o.p[q] = q == 1 ? a.p[1] + k.zr : a.p[q];
#pragma unroll
  for (int q = 0; q < 15; ++q) o.cov[q] = a.C[q];
  o.status = nh >= P.min_hits ? 0 : 1;
  return nh >= P.min_hits;
}

// The selection's claims of the wave's n tracklets that ended: the claim key
// of each goes into the owner words of its hits, four tracklets' slots in
// flight.
template <int kBlk>
__device__ __forceinline__ void fit_claim(const Bufs &B, const FitBlock<kBlk> &S, int n, int Rs) {
  static_assert(kMaxRows < 4 * 64, "a lane takes four of a tracklet's hits");
  const int lane = threadIdx.x & 63;
  const int4 *done = S.done[threadIdx.x >> 6];
  wave_lds_order();
  // the hit slots were written by other lanes of this wave
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  for (int e = 0; e < n; e += 4) {
    int4 d[4], h[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      d[q] = done[min(e + q, n - 1)];
      if (4 * lane < slot_row(d[q].w)) h[q] = reinterpret_cast<const int4 *>(B.trk_hits + (int64_t)d[q].x * Rs)[lane];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int nh = e + q < n ? slot_row(d[q].w) : 0, j = 4 * lane;
      const unsigned long long key = claim_key(nh, __int_as_float(d[q].z), d[q].w & 0xFFFFFF);
      if (j < nh) atomicMax(&B.owner[slot_hit(h[q].x, d[q].y)], key);
      if (j + 1 < nh) atomicMax(&B.owner[slot_hit(h[q].y, d[q].y)], key);
      if (j + 2 < nh) atomicMax(&B.owner[slot_hit(h[q].z, d[q].y)], key);
      if (j + 3 < nh) atomicMax(&B.owner[slot_hit(h[q].w, d[q].y)], key);
    }
  }
  wave_lds_order();  // the entries are free again
}

// Notes the lanes' tracklets that ended (fin) for the claims, n of them so far.
template <int kBlk>
__device__ __forceinline__ void fit_ended(const Bufs &B, FitBlock<kBlk> &S, bool fin, const Trk &k, int nh, float chi2,
                                          int Rs, int &n) {
  for (unsigned long long left = __ballot(fin); left;) {
    const int lane = threadIdx.x & 63, at = n + lanes_below(left);
    const bool put = (left >> lane & 1) && at < kDone;
    if (put)  // rows are as many as hits or more: a hit count has a row's size
      S.done[threadIdx.x >> 6][at] = make_int4(k.t, k.ucl, __float_as_int(chi2),
                                               (int)((uint32_t)nh << 24) | (S.head[threadIdx.x].x & 0xFFFFFF));
    const unsigned long long gone = __ballot(put);
    n += __popcll(gone);
    left &= ~gone;
    if (n == kDone) {
      fit_claim(B, S, n, Rs);
      n = 0;
    }
  }
}

// In both forms a step's memory reads (the given hit, the row's description)
// are issued in the step before, after its propagation: they overlap the
// update and the next propagation, and their registers are free meanwhile.

// ----------------------------------------------------------- few: loops ---
// Every loop leaves at its end only, and runs its arithmetic whether or not it
// has failed (what a failed tracklet computes is not used): the state then
// stays in its registers, where a way out in the middle would copy it.

// One tracklet in the wave: a loop per phase, each with nothing but its own.

// Follows a tracklet row by row from r outward (kOut) or inward.
template <int kBlk, bool kOut>
__device__ __forceinline__ void lone_follow(const Bufs &B, const ParamsDev &P, FitBlock<kBlk> &S, const Trk &k, int r,
                                           int n1, int &nh, float &chi2, int32_t *slots, KState &st, Work &w) {
  constexpr int dir = kOut ? 1 : -1;
  const int R = P.n_rows;
  int4 v = load16(B.rowtab + k.rb + max(r, 0));
  int miss = 0;
  bool go = kOut ? r < R : r >= 0;
  while (go) {
    ++w.steps;
    const bool ok = kf_step(P, st, S.rx[r]);
    int h = -1;
    float2 c = make_float2(0.0f, 0.0f);
    if (ok) h = kf_search<4>(B, P, row_bins(v), st, k.zr, w.cands, c);
    v = load16(B.rowtab + k.rb + max(r + dir, 0));
    w.tests += h >= 0 ? 1u : 0u;
    KMeas m;
    const bool pos = kf_meas(P, st, c.x, c.y - k.zr, m);
    ++miss;
    if (h >= 0 && pos && m.chi2 <= P.pick_chi2) {
      kf_gain(st, m);
      ++w.updates;
      S.aux.save(st);
      const int32_t sv = slot_enc(h, k.ucl, r);
      if (kOut) {
        S.slot.at(nh) = sv;
        if ((nh & kGM) == kGM) S.slot.flush(slots, nh);
      } else {
        chi2 = chi2 + m.chi2;
        fit_slot_in(S, n1, nh, slots, sv);
      }
      ++nh;
      miss = 0;
    }
    r += dir;
    go = ok && miss < P.max_miss && (kOut ? r < R : r >= 0);
  }
}

template <int kBlk>
__device__ __forceinline__ bool lone_tracklet(const Bufs &B, const ParamsDev &P, FitBlock<kBlk> &S, int pos, Trk &k,
                                             int &nh, float &chi2, Work &w) {
  KState st;
  int32_t sv;
  fit_start(P, S, fit_read(B, P, S.rx, pos), k, st);
  int32_t *slots = B.trk_hits + (int64_t)k.t * slot_stride(P.n_rows);
  const int r0 = k.r - 1;
  nh = 1;
  bool ok, go;
  KMeas m;
  // the chain
  do {
    ok = kf_step(P, st, S.rx[r0 + nh]);
    w.updates += ok ? 1u : 0u;
    const float2 c = hit_yz(k.v);
    const int hx = max(k.hx, 0);
    k.v = load16(B.yz + hx);
    const int hy = B.upc[hx];
    ok = kf_meas(P, st, c.x, c.y - k.zr, m) && ok;
    kf_gain(st, m);
    S.slot.at(nh) = slot_enc(k.hn, k.ucl, r0 + nh);
    if ((nh & kGM) == kGM) S.slot.flush(slots, nh);
    ++nh;
    go = ok && k.hx >= 0;
    k.hn = k.hx;
    k.hx = hy;
  } while (go);
  w.steps += nh - 1;
  if (ok) {
    S.aux.save(st);
    lone_follow<kBlk, true>(B, P, S, k, r0 + nh, 0, nh, chi2, slots, st, w);
    const int n1 = nh;
    fit_turn(B, P, S, k, n1, slots, st);
    // inward through the pass-1 hits, the outermost without a step
    int j = n1 - 1;
    sv = S.slot.at(j);
    k.v = load16(B.yz + slot_hit(sv, k.ucl));
    for (bool first = true;; first = false) {
      ok = true;
      if (!first) ok = kf_step(P, st, S.rx[slot_row(sv)]);
      w.updates += ok ? 1u : 0u;
      const float2 c = hit_yz(k.v);
      const bool fill = (j & 3) == 3 && j > 3;
      int4 q4;
      if (fill) q4 = reinterpret_cast<const int4 *>(slots)[(j >> 2) - 1];
      sv = S.slot.at(j - 1);
      k.v = load16(B.yz + (j > 0 ? slot_hit(sv, k.ucl) : 0));
      ok = kf_meas(P, st, c.x, c.y - k.zr, m) && ok;
      chi2 = first ? 0.0f + m.chi2 : chi2 + m.chi2;
      kf_gain(st, m);
      if (fill) S.slot.v[((j >> 2) - 1) & 1][threadIdx.x] = q4;
      --j;
      if (!(ok && j >= 0)) break;
    }
    w.steps += n1 - 2 - j;
    if (ok) {
      S.aux.save(st);
      lone_follow<kBlk, false>(B, P, S, k, r0 - 1, n1, nh, chi2, slots, st, w);
      return fit_done(B, P, S, k, n1, nh, chi2, slots);
    }
  }
  fit_failed(B, S, k.t);
  return false;
}

// Several tracklets in the wave: a loop per pass, its steps to given hits and to
// searched ones in one body, so that a pass takes the wave at most as many
// iterations as there are rows; with loops per phase it takes the longest
// chain's and the longest search's.  34 thousand tracklets, 16 to a wave: 0.90
// ms by phases, 0.70 by passes; 1.7 thousand, one to a wave: 0.52 and 0.60.
template <int kBlk>
__device__ __forceinline__ bool few_tracklet(const Bufs &B, const ParamsDev &P, FitBlock<kBlk> &S, int pos, Trk &k,
                                             int &nh, float &chi2, Work &w) {
  const int R = P.n_rows;
  KState st;
  fit_start(P, S, fit_read(B, P, S.rx, pos), k, st);
  int32_t *slots = B.trk_hits + (int64_t)k.t * slot_stride(R);
  const int r0 = k.r - 1;
  nh = 1;
  bool given = true, failed = false, go;
  int miss = 0;
  KMeas m;
  // outward: the chain's hits, then a search in each row
  do {
    const bool ok = kf_step(P, st, S.rx[k.r]);
    ++w.steps;
    int h = k.hn;
    float2 c = hit_yz(k.v);
    if (!given) {
      h = -1;
      if (ok) h = kf_search<4>(B, P, row_bins(k.v), st, k.zr, w.cands, c);
      w.tests += h >= 0 ? 1u : 0u;
    }
    const int hx = given ? k.hx : -1;
    k.v = load16(hx >= 0 ? (const void *)(B.yz + hx) : (const void *)(B.rowtab + k.rb + min(k.r + 1, R)));
    const int hy = B.upc[max(hx, 0)];
    const bool pos_def = kf_meas(P, st, c.x, c.y - k.zr, m);
    const bool upd = pos_def && (given ? ok : h >= 0 && m.chi2 <= P.pick_chi2);
    w.updates += (given ? ok : upd) ? 1u : 0u;
    failed = given && !upd;
    ++miss;
    if (upd) {
      kf_gain(st, m);
      S.slot.at(nh) = slot_enc(h, k.ucl, k.r);
      if ((nh & kGM) == kGM) S.slot.flush(slots, nh);
      ++nh;
      miss = 0;
      if (hx < 0) S.aux.save(st);
    }
    k.hn = hx;
    k.hx = hy;
    given = hx >= 0;
    ++k.r;
    go = given ? !failed : !failed && ok && miss < P.max_miss && k.r < R;
  } while (go);
  if (failed) {
    fit_failed(B, S, k.t);
    return false;
  }
  const int n1 = nh;
  fit_turn(B, P, S, k, n1, slots, st);
  // inward: the pass-1 hits, the outermost without a step, then a search in
  // each row below the chain
  int j = n1 - 1;
  int32_t sv = S.slot.at(j);
  k.v = load16(B.yz + slot_hit(sv, k.ucl));
  k.r = slot_row(sv);
  chi2 = 0.0f;
  given = true;
  do {
    bool ok = true;
    if (j != n1 - 1) {
      ok = kf_step(P, st, S.rx[k.r]);
      ++w.steps;
    }
    int h = -1;
    float2 c = hit_yz(k.v);
    if (!given) {
      if (ok) h = kf_search<4>(B, P, row_bins(k.v), st, k.zr, w.cands, c);
      w.tests += h >= 0 ? 1u : 0u;
    }
    const bool fill = given && (j & 3) == 3 && j > 3;
    int4 q4;
    if (fill) q4 = reinterpret_cast<const int4 *>(slots)[(j >> 2) - 1];
    sv = S.slot.at(j - 1);
    const bool more = given && j > 0;
    const int rn = more ? slot_row(sv) : k.r - 1;
    k.v = load16(more ? (const void *)(B.yz + slot_hit(sv, k.ucl)) : (const void *)(B.rowtab + k.rb + max(rn, 0)));
    const bool pos_def = kf_meas(P, st, c.x, c.y - k.zr, m);
    const bool upd = pos_def && (given ? ok : h >= 0 && m.chi2 <= P.pick_chi2);
    w.updates += (given ? ok : upd) ? 1u : 0u;
    failed = given && !upd;
    ++miss;
    if (upd) {
      kf_gain(st, m);
      chi2 = chi2 + m.chi2;
      if (!given) {
        fit_slot_in(S, n1, nh, slots, slot_enc(h, k.ucl, k.r));
        ++nh;
      }
      miss = 0;
      if (!more) S.aux.save(st);
    }
    if (fill) S.slot.v[((j >> 2) - 1) & 1][threadIdx.x] = q4;
    --j;
    given = more;
    k.r = rn;
    go = given ? !failed : !failed && ok && miss < P.max_miss && k.r >= 0;
  } while (go);
  if (failed) {
    fit_failed(B, S, k.t);
    return false;
  }
  return fit_done(B, P, S, k, n1, nh, chi2, slots);
}

template <int kBlk>
__device__ __forceinline__ void fit_few(const Bufs &B, const ParamsDev &P, RunDev &rd, FitBlock<kBlk> &S, Work &w) {
  const int lane = threadIdx.x & 63;
  int lo, hi, ended = 0;
  few_share(rd.n_trk, lo, hi);
  for (int i = lo; i < hi; i += 64) {
    Trk k;
    int nh = 0;
    float chi2 = 0.0f;
    Work mine;
    const int pos = rd.trk0 + i + lane;
    const bool fin = i + lane < hi && (hi - i == 1 ? lone_tracklet(B, P, S, pos, k, nh, chi2, mine)
                                                   : few_tracklet(B, P, S, pos, k, nh, chi2, mine));
    if (P.kf_claims) fit_ended(B, S, fin, k, nh, chi2, slot_stride(P.n_rows), ended);
    // totals of the wave; it stepped at least as often as its longest tracklet
    w.iters += (unsigned int)wave_max_dpp((int)mine.steps);
    w.steps += wave_sum(mine.steps);
    w.cands += mine.cands;
    w.tests += wave_sum(mine.tests);
    w.updates += wave_sum(mine.updates);
  }
  if (ended) fit_claim(B, S, ended, slot_stride(P.n_rows));
}

// -------------------------------------------------- many: state machine ---
// What a lane does: nothing, steps to the chain's hits or (refit) to the
// pass-1 hits, or searches (from 0 on: the number of empty rows since the
// last hit).
enum : int { kFree = -3, kLink = -2, kBack = -1, kSearch = 0 };

// Lanes without a tracklet go along on whatever their registers hold (every
// address stays in range).
template <int kBlk>
__device__ __forceinline__ void fit_many(const Bufs &B, const ParamsDev &P, RunDev &rd, FitBlock<kBlk> &S, Work &w) {
  const int R = P.n_rows, Rs = slot_stride(R);
  const int n_trk = rd.n_trk;
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  int ahead = 0, taken = 0;  // tracklets read ahead and not started, those started before them
  int ended = 0;             // tracklets whose claims are not written
  Pool pool = pool_start(P, n_trk);
  bool told = false;  // the drain's start was recorded
  int state = kFree;
  Trk k{};
  // hits of pass 1 (0 until it ends) and so far; the refit counts j down
  int n1 = 0, nh = 0, j = 0;
  float chi2 = 0.0f;
  KState st{};
  st.p[2] = 0.5f;  // a lane that never starts asks for no general division
  for (;;) {
    const unsigned long long idle = __ballot(state == kFree);
    if (idle) {
      if (ahead == 0) {
        // the next tracklets, read by as many lanes at a time
        while (pool.next == pool.end && !pool.exhausted)
          pool_claim(P, pool, rd.kf_next, n_trk, __popcll(idle), lane);
        ahead = min(kSeeds, pool.end - pool.next);
        wave_lds_order();
        if (lane < ahead) {
          const Seed a = fit_read(B, P, S.rx, rd.trk0 + pool.next + lane);
          S.seed[wid][0][lane] = make_int4(a.t, a.u, a.ucl, a.s0);
          S.seed[wid][1][lane] = make_int4(a.hn, a.hx, __float_as_int(a.next.x), __float_as_int(a.next.y));
          S.seed[wid][2][lane] = make_int4(__float_as_int(a.y), __float_as_int(a.z), __float_as_int(a.sn),
                                           __float_as_int(a.p3));
          S.seed_head[wid][lane] = a.head;
        }
        wave_lds_order();
        pool.next += ahead;
        taken = 0;
      }
      if (ahead) {
        const int take = min(__popcll(idle), ahead);
        const int rank = lanes_below(idle);
        if (state == kFree && rank < take) {
          const int4 a = S.seed[wid][0][taken + rank], b = S.seed[wid][1][taken + rank],
                     c = S.seed[wid][2][taken + rank];
          fit_start(P, S,
                    Seed{a.x, a.y, a.z, a.w, b.x, b.y, __int_as_float(c.x), __int_as_float(c.y), __int_as_float(c.z),
                         __int_as_float(c.w), make_float2(__int_as_float(b.z), __int_as_float(b.w)),
                         S.seed_head[wid][taken + rank]},
                    k, st);
          nh = 1;
          n1 = 0;
          state = kLink;
        }
        taken += take;
        ahead -= take;
      } else {
        if (idle == ~0ull) break;
        if (!told) {
          told = true;
          if (lane == 0) atomicMin(&rd.kf_t_drain, (unsigned long long)__builtin_amdgcn_s_memrealtime());
        }
      }
    }
    // ---- the step: one propagation, one search or the given hit, one update
    const bool link = state == kLink, back = state == kBack, given = link | back;
    const bool inside = k.r >= 0 && k.r < R;
    const bool prop = given ? !(back && j == n1 - 1) : state >= kSearch && inside;
    ++w.iters;
    w.steps += __popcll(__ballot(prop));
    bool ok = true;
    if (!(back && j == n1 - 1)) ok = kf_step(P, st, S.rx[min(max(k.r, 0), R)]);
    int h = k.hn;
    float2 c = hit_yz(k.v);
    bool upd = given & ok;
    const bool search = prop && !given && ok;
    if (search) {
      h = kf_search<8>(B, P, row_bins(k.v), st, k.zr, w.cands, c);
      upd = h >= 0;
    }
    w.tests += __popcll(__ballot(search && upd));
    // reads of the next step: a hit, or a row's description (also of the
    // first row after the chain or the refit)
    const bool out = n1 == 0;
    int32_t *const slots = B.trk_hits + (int64_t)k.t * Rs;
    const bool fill = back && (j & 3) == 3 && j > 3;
    int4 q4;
    if (fill) q4 = reinterpret_cast<const int4 *>(slots)[(j >> 2) - 1];
    const int32_t vx = S.slot.at(j - 1);  // refit: slot j - 1
    const int hx = link ? k.hx : back && j > 0 ? slot_hit(vx, k.ucl) : -1;
    const int rn = min(max(k.r + (out ? 1 : -1), 0), R);
    k.v = load16(hx >= 0 ? (const void *)(B.yz + hx) : (const void *)(B.rowtab + k.rb + rn));
    const int hy = B.upc[link ? max(hx, 0) : 0];
    if (upd) {
      KMeas m;
      upd = kf_meas(P, st, c.x, c.y - k.zr, m) && (given || m.chi2 <= P.pick_chi2);
      if (upd) {
        chi2 = chi2 + m.chi2;
        kf_gain(st, m);
      }
    }
    w.updates += __popcll(__ballot(given ? ok : upd));
    if (fill) S.slot.v[((j >> 2) - 1) & 1][tid] = q4;
    // ---- bookkeeping
    bool fin = false;
    if (upd) {
      bool save = !given;
      if (!back) {
        const int32_t sv = slot_enc(h, k.ucl, k.r);
        if (out) {
          S.slot.at(nh) = sv;
          if ((nh & kGM) == kGM) S.slot.flush(slots, nh);
        } else {
          fit_slot_in(S, n1, nh, slots, sv);
        }
        ++nh;
        k.r += out ? 1 : -1;
      } else if (--j >= 0) {
        k.r = slot_row(vx);
      } else {
        --k.r;
      }
      if (link) {
        k.hn = k.hx;
        k.hx = hy;
        save = hx < 0;  // the chain's last hit
      } else if (back) {
        save = j < 0;
      }
      if (save) {
        S.aux.save(st);
        state = kSearch;
      }
    } else if (given) {
      fit_failed(B, S, k.t);
      state = kFree;
    } else if (state >= kSearch) {
      if (search && ++state < P.max_miss) {
        k.r += out ? 1 : -1;
      } else if (out) {
        fit_turn(B, P, S, k, nh, slots, st);
        n1 = nh;
        j = n1 - 1;
        chi2 = 0.0f;
        const int32_t sv = S.slot.at(j);
        k.v = load16(B.yz + slot_hit(sv, k.ucl));
        k.r = slot_row(sv);
        state = kBack;
      } else {
        fin = fit_done(B, P, S, k, n1, nh, chi2, slots);
        state = kFree;
      }
    }
    if (P.kf_claims) fit_ended(B, S, fin, k, nh, chi2, Rs, ended);
  }
  if (ended) fit_claim(B, S, ended, Rs);
}

template <int kBlk>
__global__ __launch_bounds__(kBlk, 4) void k_kf(Bufs B, ParamsDev P, int run) {
  __shared__ FitBlock<kBlk> S;
  RunDev &rd = B.runs[run];
  if (threadIdx.x == 0) S.steps = S.cands = S.tests = S.updates = S.iters = 0;
  for (int i = threadIdx.x; i <= kMaxRows; i += blockDim.x) S.rx[i] = i < P.n_rows ? B.row_x[i] : 0.0f;
  __syncthreads();
  const unsigned long long t_start = __builtin_amdgcn_s_memrealtime();
  Work w;
  const bool few = rd.n_trk <= kFewMax && !P.kf_xcd;
  if (few)
    fit_few(B, P, rd, S, w);
  else
    fit_many(B, P, rd, S, w);
  if (w.iters) {
    const unsigned int cands = wave_sum(w.cands);
    if ((threadIdx.x & 63) == 0) {
      atomicAdd(&S.steps, w.steps);
      atomicAdd(&S.cands, cands);
      atomicAdd(&S.tests, w.tests);
      atomicAdd(&S.updates, w.updates);
      atomicAdd(&S.iters, w.iters);
    }
  }
  __syncthreads();
  if (threadIdx.x != 0 || S.iters == 0) return;
  atomicAdd(&rd.kf_steps, (unsigned long long)S.steps);
  atomicAdd(&rd.kf_cands, (unsigned long long)S.cands);
  atomicAdd(&rd.kf_tests, (unsigned long long)S.tests);
  atomicAdd(&rd.kf_updates, (unsigned long long)S.updates);
  atomicAdd(&rd.kf_iters, (unsigned long long)S.iters);
  atomicMin(&rd.kf_t_start, t_start);
  if (few) atomicMin(&rd.kf_t_drain, t_start);  // nothing is left to claim
  atomicMax(&rd.kf_t_end, (unsigned long long)__builtin_amdgcn_s_memrealtime());
}

// ------------------------------------------------------------ launchers ---
// Compute units and resident fit blocks per CU of the current device, for
// each block size; queried once per device (contexts on several host threads
// launch concurrently, hence the lock).
struct KfOccupancy {
  int cus = 1;
  int per[3] = {};  // 64, 128, 256 threads
};

static const KfOccupancy &kf_occupancy() {
  static std::mutex mu;
  static std::map<int, KfOccupancy> cache;
  int dev = 0;
  (void)hipGetDevice(&dev);
  std::lock_guard<std::mutex> lock(mu);
  auto it = cache.find(dev);
  if (it != cache.end()) return it->second;
  KfOccupancy o;
  int cus = 0;
  (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&o.per[0], k_kf<64>, 64, 0);
  (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&o.per[1], k_kf<128>, 128, 0);
  (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&o.per[2], k_kf<256>, 256, 0);
  o.cus = std::max(1, cus);
  for (int &b : o.per) b = std::max(1, b);
  return cache.emplace(dev, o).first->second;
}

hipError_t launch_kf(const Bufs &B, const ParamsDev &P, int run, const RunHost &h, hipStream_t s) {
  if (P.kf_rows > 0) return launch_kf_rows(B, P, run, h, s);
  if (h.trk_cap <= 0) return hipSuccess;
  // at most the resident capacity of the chip, and enough waves to give few
  // tracklets a wave each; block sizes 64, 128 (default) or 256 threads.  Four
  // waves share a SIMD, by registers (128) and by LDS.
  const int blk = kf_block_of(P);
  const int bi = blk == 64 ? 0 : blk == 256 ? 2 : 1;
  const KfOccupancy &o = kf_occupancy();
  const int per = o.per[bi];
  const int64_t cap = (int64_t)o.cus * (P.kf_blocks_per_cu > 0 ? std::min(P.kf_blocks_per_cu, per) : per);
  const int64_t need = std::max<int64_t>(((int64_t)h.trk_cap + blk - 1) / blk,
                                         std::min<int64_t>(h.trk_cap, kFewWaves) * 64 / blk + 1);
  const int g = (int)std::min(cap, need);
  if (blk == 64)
    k_kf<64><<<g, 64, 0, s>>>(B, P, run);
  else if (blk == 256)
    k_kf<256><<<g, 256, 0, s>>>(B, P, run);
  else
    k_kf<128><<<g, 128, 0, s>>>(B, P, run);
  return hipGetLastError();
}

}  // namespace tpcca
