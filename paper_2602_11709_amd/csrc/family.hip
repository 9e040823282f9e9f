// Families of symmetry-equivalent reflections in each merged peak (paper,
// Section 2: the grouping of symmetry-equivalent reflections is one of the
// steps moved to compiled code; Section 3's example output lists per peak its
// families, each with a multiplicity).
//
// Two reflections of a peak belong to one family when
//   indices rule: their absolute index values are equal as multisets, in the
//     form (h, k, l), or (h, k, -(h + k), l) on a hexagonal lattice;
//   lattice rule: a point operation M of the lattice (entries in {-1, 0, 1},
//     M^T G* M = G*) maps one onto the other, hkl -> M hkl.
// Both are class invariants of a key: the sorted absolute values, or the
// lexicographically largest image M hkl over the lattice's operations (an
// orbit has one largest member).  Members are taken in the peak's member
// order; a member whose key matches an existing family joins it, otherwise
// it opens the next family.  A family's label is its lexicographically
// largest member, its multiplicity the number of its members.
//
// A crystal whose peaks hold few members (triclinic: Friedel pairs) takes a
// thread per peak.  The others take a lane per member: a wavefront owns a
// stretch of kStretch positions of the crystal's sorted reflections and takes
// the peaks that begin there, as many whole peaks at a time as fit its 64
// lanes; each lane forms its member's key, the lanes of a peak compare keys
// through LDS, the first lane of each key leads its family, and a family's
// number is its leader's rank among the peak's leaders.  A larger peak (cubic
// coincidences, wide tolerances) takes the wavefront alone, up to four members
// a lane; one of more than kBigPeak members is walked by one lane, keeping its
// families in the peak's own stretch of the output arrays, in place: family f
// of a peak is created by a member at position >= f, so the slot holding the
// family's key (and later its label) never holds anything still needed.
//
// Bound by dependent loads (first, perm, indices) for peaks of two members and
// by the key's up to 48 operations for symmetric cells.  One thread per peak
// for every crystal left the 48 x 48 operations of a cubic peak to one lane and
// a crystal's hundred peaks to one block:
//   300 cells of the six crystal systems, lattice rule: 640 -> 51 us
//   1024 triclinic cells (1.05 M peaks): 32 -> 31 us (a lane per member: 37)
// Blocks of 256 threads (four times the positions per wavefront) took 71 us
// on the first; fewer than eight wavefronts a SIMD 38 us on the second.
#include "xrd_internal.h"

namespace xrd {

namespace {

constexpr int kThreads = 1024;
constexpr int64_t kKeyBias = (int64_t)1 << 20;  // |M hkl| entries stay below 2^20

__device__ __forceinline__ void sort2(uint32_t &a, uint32_t &b) {
  const uint32_t lo = a < b ? a : b, hi = a < b ? b : a;
  a = lo;
  b = hi;
}

__device__ __forceinline__ uint64_t index_key(int h, int k, int l, bool hex) {
  uint32_t a = (uint32_t)abs(h), b = (uint32_t)abs(k), c = (uint32_t)abs(l), d = hex ? (uint32_t)abs(h + k) : 0u;
  // sorting network on four values (the fourth is 0 in the 3-index form, which
  // leaves the multiset comparison of the other three unchanged)
  sort2(a, b);
  sort2(c, d);
  sort2(a, c);
  sort2(b, d);
  sort2(b, c);
  return ((uint64_t)a << 48) | ((uint64_t)b << 32) | ((uint64_t)c << 16) | (uint64_t)d;
}

__device__ __forceinline__ uint64_t pack_hkl(int64_t h, int64_t k, int64_t l) {
  return ((uint64_t)(h + kKeyBias) << 42) | ((uint64_t)(k + kKeyBias) << 21) | (uint64_t)(l + kKeyBias);
}

__device__ __forceinline__ uint64_t image_key(int h, int k, int l, uint32_t m) {
  int v[3];
#pragma unroll
  for (int r = 0; r < 3; ++r) {
    const int m0 = (int)((m >> (6 * r)) & 3u) - 1, m1 = (int)((m >> (6 * r + 2)) & 3u) - 1,
              m2 = (int)((m >> (6 * r + 4)) & 3u) - 1;
    v[r] = __mul24(m0, h) + __mul24(m1, k) + __mul24(m2, l);
  }
  return pack_hkl(v[0], v[1], v[2]);
}

__device__ __forceinline__ uint64_t lattice_key(int h, int k, int l, const FamOps &fo) {
  uint64_t best = 0;
  // four operations a round while there are four, their loads (uniform over
  // the wavefront) in flight together
  int o = 0;
  for (; o + 4 <= fo.n_ops; o += 4) {
    uint32_t op[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) op[e] = fo.op[o + e];
#pragma unroll
    for (int e = 0; e < 4; ++e) best = max(best, image_key(h, k, l, op[e]));
  }
  for (; o < fo.n_ops; ++o) best = max(best, image_key(h, k, l, fo.op[o]));
  return best;
}

__device__ __forceinline__ uint64_t key_of(int h, int k, int l, bool lattice, const FamOps &fo) {
  return lattice ? lattice_key(h, k, l, fo) : index_key(h, k, l, fo.hex != 0);
}

// The general walk over peak p's members (any number of families).
__device__ void families_in_place(int64_t p, const FamOps &fo, bool lattice, const int64_t *__restrict__ first,
                                  const int32_t *__restrict__ mult, const int64_t *__restrict__ perm,
                                  const int16_t *__restrict__ hh, const int16_t *__restrict__ kk,
                                  const int16_t *__restrict__ ll, int32_t *__restrict__ n_fam,
                                  int32_t *__restrict__ fam_of, int64_t *__restrict__ fam_label,
                                  int32_t *__restrict__ fam_mult) {
  const int64_t b = first[p];
  const int32_t m = mult[p];
  // pass 1: family of every member; keys of the open families at b + f
  int32_t nf = 0;
  for (int32_t i = 0; i < m; ++i) {
    const int64_t r = perm[b + i];
    const uint64_t key = key_of(hh[r], kk[r], ll[r], lattice, fo);
    int32_t f = 0;
    while (f < nf && (uint64_t)fam_label[b + f] != key) ++f;
    if (f == nf) {
      fam_label[b + nf] = (int64_t)key;
      fam_mult[b + nf] = 0;
      ++nf;
    }
    fam_of[b + i] = f;
    fam_mult[b + f] += 1;
  }
  // pass 2: labels (the keys are no longer needed)
  int32_t seen = 0;
  for (int32_t i = 0; i < m; ++i) {
    const int64_t r = perm[b + i];
    const int32_t f = fam_of[b + i];
    if (f == seen) {
      fam_label[b + f] = r;
      ++seen;
    } else {
      const int64_t c = fam_label[b + f];
      if (pack_hkl(hh[r], kk[r], ll[r]) > pack_hkl(hh[c], kk[c], ll[c])) fam_label[b + f] = r;
    }
  }
  n_fam[p] = nf;
}

constexpr int kStretch = kSortChunk / (kThreads / 64);  // positions of a wavefront
constexpr int kBigPeak = 256;                           // members of a peak compared in LDS

// A wavefront's members in LDS: keys, lexicographic ranks of the indices,
// and the leaders of a peak of more than 64.
struct FamLds {
  uint64_t key[kBigPeak + 4], hkl[kBigPeak + 4];
  uint64_t lead[kBigPeak / 64];
  uint32_t start[2];
};

__device__ __forceinline__ void fam_wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Smallest i in [lo, hi] with a[i] >= target (a ascending; hi if none), by
// 64 probes a round.
__device__ __forceinline__ int64_t wave_lower_bound(const int64_t *__restrict__ a, int64_t lo, int64_t hi,
                                                    int64_t target, int lane) {
  while (lo < hi) {
    const int64_t stride = (hi - lo + 63) / 64, i = lo + lane * stride;
    const int nb = __popcll(__ballot(i < hi && a[i] < target));  // the probes below form a prefix
    if (nb == 0) return lo;
    const int64_t last = lo + (int64_t)(nb - 1) * stride;
    hi = min(hi, last + stride);
    lo = last + 1;
  }
  return lo;
}

// What U members of a peak of m, with keys mine[], find: their family's leader
// and, for a leader, the family's size and the member of its label.  Every
// member's key and rank is read once for all U, four at a time (the arrays
// hold whole groups of four; entries past m match no member).
template <int U>
struct FamFound {
  int lead[U], count[U], label[U];
};
template <int U>
__device__ __forceinline__ FamFound<U> fam_scan(const uint64_t *key, const uint64_t *hkl, int m,
                                                const uint64_t (&mine)[U]) {
  FamFound<U> r;
  uint64_t best[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    r.lead[u] = m;
    r.count[u] = r.label[u] = 0;
    best[u] = 0;
  }
  for (int j0 = 0; j0 < m; j0 += 4) {
    uint64_t k[4], h[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      k[v] = key[j0 + v];
      h[v] = hkl[j0 + v];
    }
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int j = j0 + v;
        const bool same = k[v] == mine[u] && j < m, top = same && h[v] > best[u];
        r.lead[u] = same ? min(r.lead[u], j) : r.lead[u];
        r.count[u] += same ? 1 : 0;
        r.label[u] = top ? j : r.label[u];
        best[u] = top ? h[v] : best[u];
      }
  }
  return r;
}

// Peaks of a few members (a triclinic crystal's are Friedel pairs): a thread
// each, walking its members in order with up to kRegFam families (key, label,
// count) in registers; a peak with more is redone by the general walk.
constexpr int kRegFam = 4;
// most members a peak has on average to be walked this way: below the 8 of an
// orthorhombic general reflection, above a triclinic crystal's 2 and a
// monoclinic one's 4, whose threads still have many peaks to share
constexpr int kFewMembers = 4;
__device__ __forceinline__ void families_small(int64_t p0, int64_t p1, const FamOps &fo, bool lattice,
                                               const int64_t *__restrict__ first, const int32_t *__restrict__ mult,
                                               const int64_t *__restrict__ perm, const int16_t *__restrict__ hh,
                                               const int16_t *__restrict__ kk, const int16_t *__restrict__ ll,
                                               int32_t *__restrict__ n_fam, int32_t *__restrict__ fam_of,
                                               int64_t *__restrict__ fam_label, int32_t *__restrict__ fam_mult) {
  for (int u = 0; u < kSortChunk / kThreads; ++u) {
    const int64_t p = p0 + u * kThreads + threadIdx.x;
    if (p >= p1) break;
    const int64_t b = first[p];
    const int32_t m = mult[p];
    uint64_t fk[kRegFam] = {}, lab[kRegFam] = {};
    int64_t li[kRegFam] = {};
    int32_t cnt[kRegFam] = {};
    int32_t nf = 0;
    bool spill = false;
    for (int32_t i = 0; i < m; ++i) {
      const int64_t r = perm[b + i];
      const int h = hh[r], k = kk[r], l = ll[r];
      const uint64_t key = key_of(h, k, l, lattice, fo);
      const uint64_t ph = pack_hkl(h, k, l);
      int32_t f = -1;
#pragma unroll
      for (int g = 0; g < kRegFam; ++g)
        if (f < 0 && g < nf && fk[g] == key) f = g;
      if (f < 0) {
        if (nf == kRegFam) {
          spill = true;
          break;
        }
        f = nf++;
#pragma unroll
        for (int g = 0; g < kRegFam; ++g)
          if (g == f) {
            fk[g] = key;
            lab[g] = ph;
            li[g] = r;
          }
      }
#pragma unroll
      for (int g = 0; g < kRegFam; ++g)
        if (g == f) {
          cnt[g] += 1;
          if (ph > lab[g]) {
            lab[g] = ph;
            li[g] = r;
          }
        }
      fam_of[b + i] = f;
    }
    if (spill) {
      families_in_place(p, fo, lattice, first, mult, perm, hh, kk, ll, n_fam, fam_of, fam_label, fam_mult);
      continue;
    }
#pragma unroll
    for (int g = 0; g < kRegFam; ++g)
      if (g < nf) {
        fam_label[b + g] = li[g];
        fam_mult[b + g] = cnt[g];
      }
    n_fam[p] = nf;
  }
}

__global__ void __launch_bounds__(kThreads, 8) k_peak_families(
    const HChunk *__restrict__ chunks, const FamOps *__restrict__ fam_ops, const int64_t *__restrict__ peak_offset,
    const int64_t *__restrict__ first, const int32_t *__restrict__ mult, const int64_t *__restrict__ perm,
    const int16_t *__restrict__ hh, const int16_t *__restrict__ kk, const int16_t *__restrict__ ll, int rule,
    int32_t *__restrict__ n_fam, int32_t *__restrict__ fam_of, int64_t *__restrict__ fam_label,
    int32_t *__restrict__ fam_mult) {
  __shared__ FamLds s_lds[kThreads / 64];
  const int lane = threadIdx.x & 63;
  const int wid = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  FamLds &L = s_lds[wid];
  const HChunk ch = chunks[blockIdx.x];
  const int64_t p0 = peak_offset[ch.crystal], p1 = peak_offset[ch.crystal + 1];
  if (p0 >= p1) return;
  const FamOps &fo = fam_ops[ch.crystal];
  const bool lattice = rule == 1;
  const int64_t f0 = first[p0], fl = first[p1 - 1];
  if (fl - f0 <= (p1 - p0) * kFewMembers) {
    families_small(p0 + (int64_t)ch.chunk * kSortChunk, p1, fo, lattice, first, mult, perm, hh, kk, ll, n_fam, fam_of,
                   fam_label, fam_mult);
    return;
  }
  // stretches are counted from the crystal's first kept member
  const int64_t b0 = f0 + (int64_t)ch.chunk * kSortChunk + wid * kStretch;
  if (b0 > fl) return;
  int64_t p = wave_lower_bound(first, p0, p1, b0, lane);
  while (p < p1) {
    // the next 64 peaks; those of the stretch that fit in 64 positions
    const bool have = p + lane < p1;
    const int64_t f = have ? first[p + lane] : INT64_MAX;
    const int32_t m = have ? mult[p + lane] : 0;
    const int64_t base = __shfl(f, 0, 64);
    if (base >= b0 + kStretch) break;
    const bool fits = have && f < b0 + kStretch && f - base + m <= 64;
    const int nfit = __popcll(__ballot(fits));  // a prefix: the ends ascend
    if (nfit > 0) {
      if (lane < 2) L.start[lane] = 0;
      fam_wave_sync();
      const int at = (int)(f - base);
      if (fits) atomicOr(&L.start[at >> 5], 1u << (at & 31));
      fam_wave_sync();
      const uint64_t starts = (uint64_t)L.start[0] | ((uint64_t)L.start[1] << 32);
      const uint64_t upto = starts & (~0ull >> (63 - lane));  // bit 0 is always set
      const int s = 63 - __clzll((long long)upto), q = __popcll(upto) - 1;
      const int mq = __shfl(m, q, 64);
      const bool live = lane < s + mq;  // false between peaks that a threshold set apart
      uint64_t key = 0, hkl = 0;
      int64_t r = 0;
      if (live) {
        r = perm[base + lane];
        const int h = hh[r], k = kk[r], l = ll[r];
        key = key_of(h, k, l, lattice, fo);
        hkl = pack_hkl(h, k, l);
      }
      L.key[lane] = key;
      L.hkl[lane] = hkl;
      fam_wave_sync();
      const uint64_t own[1] = {key};
      const FamFound<1> w = fam_scan<1>(L.key + s, L.hkl + s, live ? mq : 0, own);
      const bool leads = live && s + w.lead[0] == lane;
      const uint64_t lead = __ballot(leads);
      const int64_t label = __shfl(r, s + w.label[0], 64);
      if (live) {
        // leaders of the peak before this member's leader
        const uint64_t mine = lead & ~((1ull << s) - 1);
        const int fam = __popcll(mine & ((1ull << (s + w.lead[0])) - 1));
        fam_of[base + lane] = fam;
        if (leads) {
          fam_label[base + s + fam] = label;
          fam_mult[base + s + fam] = w.count[0];
        }
        if (lane == s) n_fam[p + q] = __popcll(s + mq < 64 ? mine & ((1ull << (s + mq)) - 1) : mine);
      }
      fam_wave_sync();  // the keys are written again by the next round
      p += nfit;
      continue;
    }
    const int m0 = __shfl(m, 0, 64);
    if (m0 > kBigPeak) {
      if (lane == 0)
        families_in_place(p, fo, lattice, first, mult, perm, hh, kk, ll, n_fam, fam_of, fam_label, fam_mult);
      ++p;
      continue;
    }
    for (int i = lane; i < m0; i += 64) {
      const int64_t r = perm[base + i];
      const int h = hh[r], k = kk[r], l = ll[r];
      L.key[i] = key_of(h, k, l, lattice, fo);
      L.hkl[i] = pack_hkl(h, k, l);
    }
    fam_wave_sync();
    constexpr int U = kBigPeak / 64;
    uint64_t own[U];
#pragma unroll
    for (int u = 0; u < U; ++u) own[u] = L.key[min(64 * u + lane, m0 - 1)];
    const FamFound<U> w = fam_scan<U>(L.key, L.hkl, m0, own);
    int total = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint64_t lead = __ballot(64 * u + lane < m0 && w.lead[u] == 64 * u + lane);
      if (lane == 0) L.lead[u] = lead;
      total += __popcll(lead);
    }
    fam_wave_sync();
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = 64 * u + lane;
      if (i >= m0) break;
      const int ld = w.lead[u];
      int fam = __popcll(L.lead[ld >> 6] & ((1ull << (ld & 63)) - 1));
      for (int v = 0; v < (ld >> 6); ++v) fam += __popcll(L.lead[v]);
      fam_of[base + i] = fam;
      if (ld == i) {
        fam_label[base + fam] = perm[base + w.label[u]];
        fam_mult[base + fam] = w.count[u];
      }
    }
    if (lane == 0) n_fam[p] = total;
    fam_wave_sync();
    ++p;
  }
}

}  // namespace

void launch_peak_families(const HChunk *chunks, int64_t n_chunks, const FamOps *fam_ops, const int64_t *peak_offset,
                          const int64_t *first, const int32_t *mult, const int64_t *perm, const int16_t *h,
                          const int16_t *k, const int16_t *l, int rule, int32_t *n_fam, int32_t *fam_of,
                          int64_t *fam_label, int32_t *fam_mult, hipStream_t s) {
  launch_ranges(n_chunks, kThreads, [&](int64_t begin, int64_t count) {
    hipLaunchKernelGGL(k_peak_families, dim3((unsigned)count), dim3(kThreads), 0, s, chunks + begin, fam_ops,
                       peak_offset, first, mult, perm, h, k, l, rule, n_fam, fam_of, fam_label, fam_mult);
  });
}

}  // namespace xrd
