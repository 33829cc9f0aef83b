// One sequence's route step (Eq. 1; Algorithm 1 "Given" and steps 5-6;
// greedy verification, Section 2 "Preliminaries"): the accepted prefix, the row
// descriptors and the new lengths.  One wavefront takes a sequence's window in
// the route kernel and in the F product's launch, which can carry it as extra
// workgroups (the F product itself does not read the descriptors then); a
// whole workgroup takes a window of many rows.
#pragma once

#include "co_kernels.h"
#include "co_store.h"

namespace co {

// m = first index where draft and target disagree (B if none), or, with
// accept decisions, the first rejected position; every lane returns m
__device__ __forceinline__ int route_accepted(const RouteArgs& a, int s, int lane) {
  const int B = a.B;
  int m = B;
  if (!(a.flags & CO_ROUTE_ACCEPT_ALL)) {
    const bool bits = a.flags & CO_ROUTE_ACCEPT_BITS;
    const int32_t* dr = a.draft + static_cast<int64_t>(s) * B;
    const int32_t* tg = bits ? nullptr : a.target + static_cast<int64_t>(s) * B;
    for (int j0 = 0; j0 < B; j0 += 64) {
      const int j = j0 + lane;
      const bool diff = j < B && (bits ? dr[j] == 0 : dr[j] != tg[j]);
      const unsigned long long mask = __ballot(diff);
      if (mask) {
        m = j0 + __ffsll(static_cast<long long>(mask)) - 1;
        break;
      }
    }
  }
  return m;
}

// Whether row r (sequence r / B, window position r % B) becomes a carry row:
// a position at or after the first rejected one, outside baseline mode.  The
// same rule as route_sequence, read by one thread without the row descriptors
// (a sequence whose route step fails gets no rows at all, so its rows' F(E)
// term is never stored either way).
__device__ __forceinline__ bool route_row_carried(const RouteArgs& a, int r) {
  if (a.flags & (CO_ROUTE_ACCEPT_ALL | CO_BASELINE_MODE)) return false;
  const int s = r / a.B, j = r % a.B;
  const bool bits = a.flags & CO_ROUTE_ACCEPT_BITS;
  const int32_t* dr = a.draft + static_cast<int64_t>(s) * a.B;
  const int32_t* tg = bits ? nullptr : a.target + static_cast<int64_t>(s) * a.B;
  bool rejected = false;
  for (int i = 0; i <= j; ++i) rejected = rejected || (bits ? dr[i] == 0 : dr[i] != tg[i]);
  return rejected;
}

// The same for the rows of a tile of BM rows from m0, whose products do not wait
// for it: every lane of each wavefront loads the tokens of one of the 64 rows
// that end with the tile, and one ballot at the end tells where a row's
// sequence was first rejected.  Reaches back to the start of every sequence in
// the tile when B - 1 <= 64 - BM (ok()); longer windows take route_row_carried.
template <int BM>
struct RouteTile {
  int32_t d, t;
  __device__ static bool ok(const RouteArgs& a) { return a.B - 1 <= 64 - BM; }
  __device__ static int base(int m0) { return m0 + BM - 64; }
  __device__ void load(const RouteArgs& a, int m0, int M, int lane) {
    const int r = min(max(base(m0) + lane, 0), M - 1);
    d = a.draft[r];
    t = (a.flags & CO_ROUTE_ACCEPT_BITS) ? 0 : a.target[r];
  }
  // row r of the tile (r < M); called by whole wavefronts
  __device__ bool carried(const RouteArgs& a, int m0, int r) const {
    const bool rej = (a.flags & CO_ROUTE_ACCEPT_BITS) ? d == 0 : d != t;
    const uint64_t mask = __ballot(rej);
    const int b = base(m0), lo = r / a.B * a.B - b, hi = r - b;   // 0 <= lo <= hi < 64
    return ((mask >> lo) & (~0ull >> (63 - (hi - lo)))) != 0;
  }
};

// What a window cannot be routed for, before its pages are looked at.
__device__ __forceinline__ int route_length_error(const RouteArgs& a, int p0) {
  if (p0 < 0) return CO_ERR_LENGTH;
  const int64_t cap = static_cast<int64_t>(a.max_pages) * kPage;
  return static_cast<int64_t>(p0) + a.B > cap ? CO_ERR_CAPACITY : 0;
}

// Whether a page of the rows this thread takes (t, t + nt, ..) of the accepted
// ones is out of range.
__device__ __forceinline__ bool route_bad_page(const RouteArgs& a, int s, int p0, int m, int t,
                                               int nt) {
  const int32_t* pt = a.page_table + static_cast<int64_t>(s) * a.max_pages;
  bool bad = false;
  for (int j = t; j < m; j += nt) {
    const int page = pt[(p0 + j) / kPage];
    bad |= page < 0 || page >= a.num_pages;
  }
  return bad;
}

// Descriptors of rows t, t + nt, .. and (thread 0) the new lengths.
__device__ __forceinline__ void route_write(const RouteArgs& a, int s, int p0, int m, int err,
                                            int t, int nt) {
  const int B = a.B;
  const bool carry_only = a.flags & CO_ROUTE_CARRY_ONLY;
  const bool baseline = a.flags & CO_BASELINE_MODE;
  const int32_t* pt = a.page_table + static_cast<int64_t>(s) * a.max_pages;
  int32_t* pos_out = a.row_pos + static_cast<int64_t>(s) * B;
  int32_t* dst_out = a.row_dst + static_cast<int64_t>(s) * B;
  if (err) {
    for (int j = t; j < B; j += nt) {
      pos_out[j] = p0 >= 0 ? p0 + j : 0;
      dst_out[j] = kSkip;
    }
    if (t == 0) {
      a.accept_len[s] = 0;
      set_status(a.status, err);
    }
    return;
  }

  for (int j = t; j < B; j += nt) {
    const int pos = p0 + j;
    int32_t dst = kSkip;
    if (j < m) {
      if (!carry_only) dst = pt[pos / kPage] * kPage + pos % kPage;
    } else if (!baseline) {
      dst = -1 - (j - m);
    }
    pos_out[j] = pos;
    dst_out[j] = dst;
  }
  if (t == 0) {
    a.accept_len[s] = m;
    a.ctx_len[s] = p0 + m;
    a.carry_len[s] = baseline ? 0 : B - m;
  }
}

__device__ __forceinline__ void route_sequence(const RouteArgs& a, int s, int lane) {
  const int p0 = a.ctx_len[s];
  const int m = route_accepted(a, s, lane);
  int err = route_length_error(a, p0);
  if (err == 0 && !(a.flags & CO_ROUTE_CARRY_ONLY) &&
      __any(route_bad_page(a, s, p0, m, lane, 64)))
    err = CO_ERR_PAGE_RANGE;
  route_write(a, s, p0, m, err, lane, 64);
}

}  // namespace co
