// Device-side scans of a grouped product's counts, shared by the grouped
// kernels: from a row-tile slot to its group and rows. Included INSIDE the
// kernels' namespace, after device_common.h.

__device__ __forceinline__ int64_t uniform64(int64_t v) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)v >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// Row ranges and row-tile counts of 64 consecutive groups, one per lane, as
// wave-wide inclusive prefix sums (rows_incl clamped by the caller).
template <int BM>
struct GroupChunk {
  int64_t lo, r;  // first row and row count of the lane's group
  int t, ts;      // row tiles of the lane's group, inclusive sum over the chunk
  int64_t rsum;   // rows of the whole chunk (unclamped)
  __device__ __forceinline__ void load(const GroupArgs& a, int c, int64_t row_base) {
    const int lane = threadIdx.x & 63;
    const int gi = c + lane;
    const int64_t cnt = gi < a.groups ? (int64_t)max(a.counts[gi], 0) : 0;
    int64_t p = cnt;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int64_t o = __shfl_up(p, d);
      if (lane >= d) p += o;
    }
    const int64_t hi = min(row_base + p, a.rows);
    lo = min(row_base + p - cnt, a.rows);
    r = hi - lo;
    t = (int)((r + BM - 1) / BM);
    ts = t;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int o = __shfl_up(ts, d);
      if (lane >= d) ts += o;
    }
    rsum = __shfl(p, 63);
  }
};

// Total row tiles of all groups.
template <int BM>
__device__ __forceinline__ int group_tiles_total(const GroupArgs& a, const GroupChunk<BM>& first) {
  int total = __shfl(first.ts, 63);
  int64_t row_base = min(first.rsum, a.rows);
  for (int c = 64; c < a.groups; c += 64) {
    GroupChunk<BM> k;
    k.load(a, c, row_base);
    total += __shfl(k.ts, 63);
    row_base = min(row_base + k.rsum, a.rows);
  }
  return total;
}

// Group, first row, row count and row tile of `slot`; false if the slot is
// past the last tile.
template <int BM>
__device__ __forceinline__ bool group_of_slot(const GroupArgs& a, const GroupChunk<BM>& first, int slot, int& grp,
                                              int64_t& row0, int64_t& rows_g, int& tm) {
  int tile_base = 0;
  int64_t row_base = 0;
  GroupChunk<BM> k = first;
  for (int c = 0; c < a.groups; c += 64) {
    if (c > 0) k.load(a, c, row_base);
    const uint64_t hit = __ballot(tile_base + k.ts > slot);
    if (hit) {
      const int f = __builtin_ctzll(hit);
      grp = c + f;
      row0 = __shfl(k.lo, f);
      rows_g = __shfl(k.r, f);
      tm = slot - (tile_base + __shfl(k.ts, f) - __shfl(k.t, f));
      return true;
    }
    tile_base += __shfl(k.ts, 63);
    row_base = min(row_base + k.rsum, a.rows);
  }
  return false;
}
