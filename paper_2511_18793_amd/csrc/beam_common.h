// Wave reductions and list handling shared by the decode kernels (decode_lds.h, beam_level.h).
// Included inside the library's unnamed namespace, after beam_args.h and device_common.h.
#pragma once

// A barrier that orders the workgroup's LDS accesses only: global loads and stores of the waves stay in
// flight across it.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// A copy of x that the compiler cannot trace back: what is computed from it (LDS addresses and the like)
// is formed where it is used instead of being kept in registers from the start of the kernel on.
__device__ __forceinline__ int fresh(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

// ---- small wave helpers --------------------------------------------------------------------------
template <int CTRL>
__device__ __forceinline__ float dpp_f(float x) {
  return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x), CTRL, 0xF,
                                                               0xF, true));
}
// Sum / maximum over the 16 lanes of a row (every lane gets it): rotations by 8, 4, 2, 1.
__device__ __forceinline__ float row_sum(float x) {
  x += dpp_f<0x128>(x);
  x += dpp_f<0x124>(x);
  x += dpp_f<0x122>(x);
  x += dpp_f<0x121>(x);
  return x;
}
__device__ __forceinline__ float row_max(float x) {
  x = max_of_numbers(x, dpp_f<0x128>(x));
  x = max_of_numbers(x, dpp_f<0x124>(x));
  x = max_of_numbers(x, dpp_f<0x122>(x));
  x = max_of_numbers(x, dpp_f<0x121>(x));
  return x;
}
__device__ __forceinline__ uint32_t row_sum_u(uint32_t x) {
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x128, 0xF, 0xF, true);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x124, 0xF, 0xF, true);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x122, 0xF, 0xF, true);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x121, 0xF, 0xF, true);
  return x;
}
__device__ __forceinline__ float wave_max_f(float x, int lane) {
  x = row_max(x);
  x = fmaxf(x, __uint_as_float(lane_xor<16>(__float_as_uint(x), lane)));
  return fmaxf(x, __uint_as_float(lane_xor<32>(__float_as_uint(x), lane)));
}
__device__ __forceinline__ float wave_sum_f(float x, int lane) {
  x = row_sum(x);
  x += __uint_as_float(lane_xor<16>(__float_as_uint(x), lane));
  return x + __uint_as_float(lane_xor<32>(__float_as_uint(x), lane));
}
// Inclusive prefix sum over the 64 lanes.
__device__ __forceinline__ uint32_t wave_prefix(uint32_t x) {
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, true);   // row_shr:1
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, true);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, true);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, true);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xA, 0xF, false);  // row_bcast:15
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xC, 0xF, false);  // row_bcast:31
  return x;
}
__device__ __forceinline__ int lane_rank(uint64_t mask) {   // set bits of mask below this lane
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                        __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0));
}

// ---- K best of a list, outputs ---------------------------------------------------------------------
// Calls emit(entry, place) for the entries of list[0..n) (distinct keys) whose place in descending
// order is below `most`: every entry is compared with every other one; a list of up to 512
// entries is shared by all waves (entry x part of the list).  rank: kBeamThreads words.
// Ends without a barrier; a barrier must separate it from the writes of list before it.
template <class Emit>
__device__ __forceinline__ void rank_list(const uint64_t* list, int n, int most, uint32_t* rank,
                                          int wave, int lane, Emit emit) {
  const int tid = wave * 64 + lane;
  if (n <= kBeamThreads) {
    const int nw = (n + 63) >> 6;                         // waves that hold the list once
    const int parts = nw > 0 ? kBeamWaves / nw : 0;
    const int part = nw > 0 ? wave / nw : 0;
    const int i = (wave - part * nw) * 64 + lane;
    rank[tid] = 0u;
    lds_barrier();
    if (part < parts) {
      const uint64_t mine = i < n ? list[i] : ~0ull;
      // even bounds: the list is read two keys at a time
      const int j0 = ((n * part) / parts) & ~1, j1 = part + 1 == parts ? n : ((n * (part + 1)) / parts) & ~1;
      uint32_t r = 0;
      int j = j0;
      for (; j + 4 <= j1; j += 4) {
        const ulonglong2 a = *reinterpret_cast<const ulonglong2*>(list + j);
        const ulonglong2 b = *reinterpret_cast<const ulonglong2*>(list + j + 2);
        r += (a.x > mine) + (a.y > mine) + (b.x > mine) + (b.y > mine);
      }
      for (; j < j1; ++j) r += list[j] > mine;
      if (i < n && r) atomicAdd(&rank[i], r);
    }
    lds_barrier();
    const int me = tid;
    if (me < n) {
      const int r = (int)rank[me];
      if (r < most) emit(list[me], r);
    }
  } else {
    for (int i = tid; i < n; i += kBeamThreads) {
      const uint64_t mine = list[i];
      uint32_t r = 0;
      int j = 0;
#pragma unroll 4
      for (; j + 2 <= n; j += 2) {
        const ulonglong2 a = *reinterpret_cast<const ulonglong2*>(list + j);
        r += (a.x > mine) + (a.y > mine);
      }
      if (j < n) r += list[j] > mine;
      if ((int)r < most) emit(mine, (int)r);
    }
  }
}

__device__ __forceinline__ uint64_t beam_entry(float score, int parent, uint32_t code) {
  return ((uint64_t)ordered_bits(score) << 32) | (uint32_t)~(((uint32_t)parent << 24) | code);
}
__device__ __forceinline__ int entry_parent(uint64_t e) { return (int)(~(uint32_t)e >> 24); }
__device__ __forceinline__ uint32_t entry_code(uint64_t e) { return ~(uint32_t)e & 0xFFFFFFu; }
__device__ __forceinline__ float entry_score(uint64_t e) { return unordered_bits((uint32_t)(e >> 32)); }


// ---- lists in eight parts ----
// While candidates are listed, every wave appends to a part of its own (positions from ballots: nothing
// has to come back from LDS); an entry belongs to the lane that the position falls to.
constexpr int kBeamMaxPer = 4;             // entries of a part per lane
constexpr int kPart = 64 * kBeamMaxPer;    // entries of a part
static_assert(kBeamList == kBeamWaves * kPart, "eight parts");
// Appends the entries of the lanes in `pass`; n: the part's length so far (it keeps counting once
// the part is full).
__device__ __forceinline__ void part_push(uint64_t* part, int& n, uint64_t pass, bool in, uint64_t entry) {
  const int at = n + lane_rank(pass);
  if (in && at < kPart) part[at] = entry;
  n += __popcll(pass);
}
// The lane's entries of a part of n.
__device__ __forceinline__ void part_mine(const uint64_t* part, int n, int lane, uint64_t (&mine)[kBeamMaxPer]) {
  __builtin_amdgcn_wave_barrier();                         // (LDS serves a wave in order)
#pragma unroll
  for (int u = 0; u < kBeamMaxPer; ++u) mine[u] = lane + 64 * u < n ? part[lane + 64 * u] : 0ull;
}
// Sums of the eight waves' counts (16-byte aligned in LDS; a barrier after they were written).
struct WaveCounts {
  int total, before, most;                 // all waves; the waves below this one; the largest
};
__device__ __forceinline__ WaveCounts wave_counts(const int* n, int wave) {
  const int4 a = *reinterpret_cast<const int4*>(n), b = *reinterpret_cast<const int4*>(n + 4);
  const int x[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
  WaveCounts w = {0, 0, 0};
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    w.total += x[q];
    w.before += q < wave ? x[q] : 0;
    w.most = x[q] > w.most ? x[q] : w.most;
  }
  w.total = __builtin_amdgcn_readfirstlane(w.total);
  w.before = __builtin_amdgcn_readfirstlane(w.before);
  w.most = __builtin_amdgcn_readfirstlane(w.most);
  return w;
}
__device__ __forceinline__ int count_marked(uint32_t ok) {
  int n = 0;
#pragma unroll
  for (int u = 0; u < kBeamMaxPer; ++u) n += __popcll(__ballot((ok >> u) & 1u));
  return n;
}
// Writes the marked entries to list[at ..] (every wave has read its own).
__device__ __forceinline__ void pack_marked(uint64_t* list, int at, uint32_t ok,
                                            const uint64_t (&mine)[kBeamMaxPer]) {
#pragma unroll
  for (int u = 0; u < kBeamMaxPer; ++u) {
    const bool in = (ok >> u) & 1u;
    const uint64_t bal = __ballot(in);
    if (bal == 0ull) continue;
    if (in) list[at + lane_rank(bal)] = mine[u];
    at += __popcll(bal);
  }
}
// Marks the lane's entries (of a part of n) that are in the set.
__device__ __forceinline__ uint32_t probe_mine(const SetView& set, const uint64_t* keys, int n, int lane,
                                               const uint64_t (&mine)[kBeamMaxPer]) {
  uint32_t ok = 0;
#pragma unroll 1
  for (int u = 0; u < kBeamMaxPer; ++u) {
    if (64 * u >= n) break;
    const uint64_t lo = (u & 1) ? mine[1] : mine[0], hi = (u & 1) ? mine[3] : mine[2];
    const uint64_t e = (u & 2) ? hi : lo;
    bool in = false;
    if (lane + 64 * u < n)
      in = set_probe(set, keys[entry_parent(e)] + (uint64_t)entry_code(e) * set.mult_last);
    ok |= (in ? 1u : 0u) << u;
  }
  return ok;
}
// Packs the marked entries to the front of the list (every thread has read its entries and a
// barrier has passed; s.n_valid is 0).  No barrier at the end.
template <class S, int kPer>
__device__ __forceinline__ void pack_list(S& s, uint64_t* list, uint32_t ok,
                                          const uint64_t (&mine)[kPer], int lane) {
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const bool in = (ok >> u) & 1u;
    const uint64_t bal = __ballot(in);
    if (bal == 0ull) continue;
    int at = 0;
    if (lane == 0) at = atomicAdd(&s.n_valid, __popcll(bal));
    at = __builtin_amdgcn_readfirstlane(at) + lane_rank(bal);
    if (in) list[at] = mine[u];
  }
}
