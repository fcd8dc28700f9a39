// Dedup and IDMap kernels of the sparse embedding step (gfx950).
//
// RecIS keeps a two-tier store: an IDMap from feature id to an offset and
// Blocks holding the rows ("Optimization for Memory Bound"); ids are
// deduplicated before the lookup ("ids partition").  The dedup gives the
// unique keys in first-occurrence order.  It uses no global atomics (on this
// GPU they serialise at the memory side): keys are grouped by a hash
// partition instead, so every key is counted by exactly one block in LDS.
//   k_tile_dedup     per block, consecutive tiles of 4096 occurrences: LDS
//                    dedup; one record per distinct key of a tile (key, first
//                    position and count in the tile), the tile's records in
//                    the order of their first positions; at the end the block
//                    copies its records into partition order
//   k_part_dedup     one block per partition, reading its records from every
//                    dedup block: LDS dedup (first position = min, count =
//                    sum, rank base of each record), the key's IDMap probe;
//                    the key's first record is flagged
//   k_first_sums     per tile of records: sums over the first records (keys,
//                    counts, keys not found, hot keys, backward units); the
//                    records, tile after tile, list each key once in the
//                    order of its first position
//   k_scan5          scan of those tile sums; reserves the rows of new keys
//   k_compact        unique ids in first-occurrence order, occurrence-list
//                    segments, rows; new keys claim an IDMap slot
//   k_occ_init       per occurrence: unique id (inverse), row, position in the
//                    occurrence list.  Its other blocks write the hot keys'
//                    backward units and the initial rows of the new keys
// A batch of at most kSmallIds ids on a table that need not grow takes two
// launches instead of these six: k_small_dedup and k_small_rows.
#include "device_common.h"

#include <algorithm>

namespace rs {

// ---------------------------------------------------------------------------
// open addressing (linear probing)
// ---------------------------------------------------------------------------

// Row of an encoded key, or -1 when the probe reaches an empty slot; the
// probe starts `done` slots into the key's sequence (at slot h).  Reads
// kProbeBatch consecutive slots per round trip.
__device__ inline int64_t idmap_lookup_at(const TableDev& t, unsigned long long e, uint64_t h, uint64_t done) {
  for (uint64_t probed = done; probed <= t.cap_mask; probed += kProbeBatch) {
    Slot sl[kProbeBatch];
#pragma unroll
    for (int k = 0; k < kProbeBatch; ++k) sl[k] = t.slots[(h + k) & t.cap_mask];
    int64_t r = -1;
    bool fin = false;
#pragma unroll
    for (int k = 0; k < kProbeBatch; ++k) {  // selects only: the batch stays in registers
      const bool hit = !fin && sl[k].key == e;
      const bool empty = !fin && sl[k].key == kEncEmpty;
      r = hit ? sl[k].row : r;
      fin = fin || hit || empty;
    }
    if (fin) return r;
    h = (h + kProbeBatch) & t.cap_mask;
  }
  return -1;
}

__device__ inline int64_t idmap_lookup(const TableDev& t, unsigned long long e) {
  return idmap_lookup_at(t, e, idmap_hash(e) & t.cap_mask, 0);
}

// Claim the slot of an encoded key (its own if present, else the first empty
// one on its probe sequence); returns the slot index or -1 if the table is
// full.  Reads kProbeBatch slot keys per round trip; a stale read of an
// empty slot only costs a failed compare-and-swap (slots are never emptied
// during a call, so a slot read as occupied stays occupied).
__device__ inline int64_t idmap_claim(const TableDev& t, unsigned long long e) {
  uint64_t h = idmap_hash(e) & t.cap_mask;
  for (uint64_t probed = 0; probed <= t.cap_mask; probed += kProbeBatch) {
    unsigned long long k[kProbeBatch];
#pragma unroll
    for (int q = 0; q < kProbeBatch; ++q) k[q] = t.slots[(h + q) & t.cap_mask].key;
    for (int q = 0; q < kProbeBatch; ++q) {
      const uint64_t hq = (h + q) & t.cap_mask;
      if (k[q] == e) return static_cast<int64_t>(hq);
      if (k[q] == kEncEmpty) {
        const unsigned long long old = atomicCAS(&t.slots[hq].key, kEncEmpty, e);
        if (old == kEncEmpty || old == e) return static_cast<int64_t>(hq);
      }
    }
    h = (h + kProbeBatch) & t.cap_mask;
  }
  return -1;
}

// Exclusive block scan of five values per thread at once (two barriers).
template <int NT>
__device__ inline void block_excl_scan5(const int (&v)[5], int (&ex)[5], int (&tot)[5], int (*sh)[5]) {
  const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
  int inc[5];
#pragma unroll
  for (int a = 0; a < 5; ++a) inc[a] = wave_incl_scan(v[a]);
  if (lane == kWave - 1) {
#pragma unroll
    for (int a = 0; a < 5; ++a) sh[wid][a] = inc[a];
  }
  __syncthreads();
  if (wid == 0) {  // one wave scans the per-wave totals of each value
    static_assert(NT / kWave <= kWave, "one wave scans the per-wave totals");
#pragma unroll
    for (int a = 0; a < 5; ++a) {
      const int t = lane < NT / kWave ? sh[lane][a] : 0;
      const int i2 = wave_incl_scan(t);
      if (lane < NT / kWave) sh[lane][a] = i2 - t;
      if (lane == kWave - 1) sh[NT / kWave][a] = i2;
    }
  }
  __syncthreads();
#pragma unroll
  for (int a = 0; a < 5; ++a) {
    ex[a] = sh[wid][a] + inc[a] - v[a];
    tot[a] = sh[NT / kWave][a];
  }
  __syncthreads();
}

// Slot hash of a tile's LDS table (32-bit multiplies: the 64-bit mix costs
// several times the instructions, once per id).
__device__ inline uint32_t lds_hash(unsigned long long e) {
  uint32_t x = static_cast<uint32_t>(e) ^ static_cast<uint32_t>(e >> 32) * 0x9E3779B1u;
  x = (x ^ (x >> 16)) * 0x85EBCA6Bu;
  x = (x ^ (x >> 13)) * 0xC2B2AE35u;
  return x >> 16;
}

__device__ inline uint32_t part_of(unsigned long long e, int logP) {
  return logP == 0 ? 0u : static_cast<uint32_t>(part_hash(e) >> (64 - logP));
}

// ---------------------------------------------------------------------------
// pass 1: tile dedup in LDS; one record per distinct key of a tile
// ---------------------------------------------------------------------------

// A dedup block whose records fill at most this many LDS chunks (8192
// records each) writes their partition-order copy with coalesced stores.
constexpr int kStageChunks = 4;

template <int NT>
__global__ __launch_bounds__(NT) void k_tile_dedup(const int64_t* __restrict__ values, int64_t n, Work w, int* err) {
  constexpr int TILE = NT * kDedupItems;
  constexpr int SLOTS = 2 * TILE;  // LDS hash slots (load <= 0.5)
  static_assert(TILE == kDedupTile, "tile size");
  // One LDS buffer: the hash table while the tiles are deduplicated (slot
  // keys; lmin: the key's first position in the tile, then its record
  // index; lcnt: its count), then the staging buffer of the partition-order
  // copy (one 16-byte record per slot).
  __shared__ TileRec lbuf[SLOTS];
  unsigned long long* const lkey = reinterpret_cast<unsigned long long*>(lbuf);
  unsigned int* const lmin = reinterpret_cast<unsigned int*>(lkey + SLOTS);
  unsigned int* const lcnt = lmin + SLOTS;
  __shared__ short ldense[TILE];          // the tile's distinct keys: dense index -> LDS slot
  __shared__ unsigned int lpc[kMaxParts];  // the block's records per partition
  __shared__ int sh[NT / kWave + 1];
  __shared__ int lfirst[kDedupItems * (NT / kWave) + 1];  // first occurrences per (item, wave), then their prefix
  const FrontGeom g = w.g;
  const int tid = threadIdx.x;
  const int64_t blk = blockIdx.x;
  for (int q = tid; q < g.P; q += NT) lpc[q] = 0u;
  if (blk == 0 && tid == 0) w.scal[kCScanDone] = 0;  // completion counter of this call's scan
  const int64_t t0 = blk * g.R;
  const int64_t t1 = min(t0 + g.R, g.ntiles);
  TileRec* rec = w.trec + blk * g.rcap;
  // the next tile's ids are loaded while this one is processed (n > 0:
  // indices are clamped)
  int64_t nxt[kDedupItems];
#pragma unroll
  for (int k = 0; k < kDedupItems; ++k) nxt[k] = values[min(t0 * TILE + k * NT + tid, n - 1)];
  unsigned int nrec = 0;
  for (int64_t tile = t0; tile < t1; ++tile) {
    const int64_t base = tile * TILE;
    int64_t raw[kDedupItems];
#pragma unroll
    for (int k = 0; k < kDedupItems; ++k) raw[k] = nxt[k];
    if (tile + 1 < t1) {
#pragma unroll
      for (int k = 0; k < kDedupItems; ++k) nxt[k] = values[min(base + TILE + k * NT + tid, n - 1)];
    }
    if (tile == t0) {  // later tiles find the table cleared by their predecessor
      for (int q = tid; q < SLOTS; q += NT) {
        lkey[q] = kEncEmpty;
        lmin[q] = 0xFFFFFFFFu;
        lcnt[q] = 0u;
      }
    }
    __syncthreads();
    int ls[kDedupItems];
    unsigned int lr[kDedupItems];
    // the home slots of a thread's ids are tried together, then each id that
    // met another key probes on
    unsigned long long was[kDedupItems];
#pragma unroll
    for (int k = 0; k < kDedupItems; ++k) {
      const int64_t i = base + k * NT + tid;
      const unsigned long long e = static_cast<unsigned long long>(raw[k]) ^ kSign;
      ls[k] = -1;
      if (i >= n) continue;
      if (e <= kEncTomb) {
        atomicOr(err, kErrKey);
        continue;
      }
      ls[k] = static_cast<int>(lds_hash(e) & (SLOTS - 1));
      was[k] = atomicCAS(&lkey[ls[k]], kEncEmpty, e);
    }
#pragma unroll
    for (int k = 0; k < kDedupItems; ++k) {
      lr[k] = 0;
      if (ls[k] < 0) continue;
      const unsigned long long e = static_cast<unsigned long long>(raw[k]) ^ kSign;
      unsigned int h = static_cast<unsigned int>(ls[k]);
      while (was[k] != kEncEmpty && was[k] != e) {  // at most TILE keys in twice as many slots: terminates
        h = (h + 1) & (SLOTS - 1);
        was[k] = atomicCAS(&lkey[h], kEncEmpty, e);
      }
      atomicMin(&lmin[h], static_cast<unsigned int>(base + k * NT + tid));
      lr[k] = atomicAdd(&lcnt[h], 1u);
      ls[k] = static_cast<int>(h);
    }
    __syncthreads();
    // dense list of the tile's keys in the order of their first positions:
    // the first occurrences (lmin of the slot is the position itself), ranked
    // in position order (item k of thread tid is position base + k*NT + tid:
    // item-major, then wave, then lane)
    int d;
    {
      constexpr int NW = NT / kWave;
      const int lane = tid & (kWave - 1), wid = tid / kWave;
      const uint64_t below = (1ull << lane) - 1ull;
      bool fst[kDedupItems];
      uint64_t bal[kDedupItems];
#pragma unroll
      for (int k = 0; k < kDedupItems; ++k) {
        const int64_t i = base + k * NT + tid;
        fst[k] = ls[k] >= 0 && lmin[ls[k]] == static_cast<unsigned int>(i);
        bal[k] = __ballot(fst[k]);
        if (lane == 0) lfirst[k * NW + wid] = __popcll(bal[k]);
      }
      __syncthreads();
      if (tid < kWave) {  // exclusive prefix over (item, wave) in position order: one wave's scan
        static_assert(kDedupItems * NW <= kWave, "one wave scans the (item, wave) counts");
        const int c = tid < kDedupItems * NW ? lfirst[tid] : 0;
        const int inc = wave_incl_scan(c);
        if (tid < kDedupItems * NW) lfirst[tid] = inc - c;
        if (tid == kWave - 1) lfirst[kDedupItems * NW] = inc;
      }
      __syncthreads();
#pragma unroll
      for (int k = 0; k < kDedupItems; ++k)
        if (fst[k]) ldense[lfirst[k * NW + wid] + __popcll(bal[k] & below)] = static_cast<short>(ls[k]);
      d = lfirst[kDedupItems * NW];
    }
    __syncthreads();
    // one record per distinct key (nrec + d <= the block's occurrences <= rcap)
    for (int q = tid; q < d; q += NT) {
      const int sl = ldense[q];
      const unsigned long long e = lkey[sl];
      const unsigned int part = part_of(e, g.logP);
      const unsigned int pr = atomicAdd(&lpc[part], 1u);
      rec[nrec + q] = TileRec{e, part, (pr << 12) | (lcnt[sl] - 1u)};
      lmin[sl] = nrec + static_cast<unsigned int>(q);
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kDedupItems; ++k) {
      const int64_t i = base + k * NT + tid;
      if (i >= n) continue;
      // read again only by the passes after the compaction: non-temporal
      __builtin_nontemporal_store(ls[k] < 0 ? kOccRejected : ((lmin[ls[k]] << 12) | lr[k]), &w.occ_word[i]);
    }
    nrec += static_cast<unsigned int>(d);
    __syncthreads();
    // empty the occupied slots for the next tile
    for (int q = tid; q < d; q += NT) {
      const int sl = ldense[q];
      lkey[sl] = kEncEmpty;
      lmin[sl] = 0xFFFFFFFFu;
      lcnt[sl] = 0u;
    }
  }
  if (tid == 0) w.nrec[blk] = static_cast<int>(nrec);
  // the block's records per partition and their offsets in partition order
  // (in place in lpc), then the partition-ordered copy of the records
  constexpr int PPT = kMaxParts / NT;
  int c[PPT];
  int loc = 0;
#pragma unroll
  for (int j = 0; j < PPT; ++j) {
    const int q = tid * PPT + j;
    c[j] = q < g.P ? static_cast<int>(lpc[q]) : 0;
    loc += c[j];
  }
  int tot;
  int run = block_excl_scan<NT>(loc, sh, tot);
#pragma unroll
  for (int j = 0; j < PPT; ++j) {
    const int q = tid * PPT + j;
    if (q < g.P) {
      w.pcnt[blk * g.P + q] = c[j];
      w.poff[blk * g.P + q] = run;
      lpc[q] = static_cast<unsigned int>(run);
    }
    run += c[j];
  }
  __syncthreads();
  TileRec* srt = w.srec + blk * g.rcap;
  const unsigned int src0 = static_cast<unsigned int>(blk * g.rcap);
  constexpr int U8 = 8;  // records in flight per thread
  // Record j goes to position lpc[partition] + its rank in the partition.
  // A block of at most kStageChunks chunks of SLOTS records assembles each
  // chunk in LDS (every pass reads all of the block's records again) and
  // writes it out with coalesced full-line stores; a larger block scatters
  // the records (runs of a few 16-byte records per partition: partial-line
  // writes, costly once the copies outgrow the memory-side cache).
  const unsigned int chunks = (nrec + SLOTS - 1) / SLOTS;
  const bool staged = chunks <= static_cast<unsigned int>(kStageChunks);
  for (unsigned int ch = 0; ch < (staged ? chunks : 1u); ++ch) {
    const unsigned int o0 = ch * SLOTS;
    const unsigned int o1 = min(o0 + static_cast<unsigned int>(SLOTS), nrec);
    for (unsigned int j0 = tid; j0 < nrec; j0 += U8 * NT) {
      TileRec r[U8];
#pragma unroll
      for (int u = 0; u < U8; ++u) {
        const unsigned int j = j0 + u * NT;
        if (j < nrec) r[u] = rec[j];
      }
#pragma unroll
      for (int u = 0; u < U8; ++u) {
        const unsigned int j = j0 + u * NT;
        if (j >= nrec) continue;
        const unsigned int o = lpc[r[u].src] + (r[u].meta >> 12);
        const TileRec x{r[u].key, src0 + j, r[u].meta & 0xFFFu};
        if (!staged) srt[o] = x;
        else if (o >= o0 && o < o1) lbuf[o - o0] = x;
      }
    }
    if (staged) {
      __syncthreads();
      for (unsigned int o = o0 + tid; o < o1; o += NT) srt[o] = lbuf[o - o0];
      __syncthreads();  // the next chunk reuses the buffer
    }
  }
}

// ---------------------------------------------------------------------------
// pass 2: one block per partition: LDS dedup of its records, IDMap probe
// ---------------------------------------------------------------------------

// Resolve a probe batch read at the key's home slot; continue the probe if
// the batch neither holds the key nor an empty slot.
__device__ inline int64_t resolve_probe(const TableDev& t, unsigned long long e, uint64_t h,
                                        const Slot (&pb)[kProbeBatch]) {
  int64_t r = -1;
  bool done = false;
#pragma unroll
  for (int q = 0; q < kProbeBatch; ++q) {  // selects only: the batch stays in registers
    const bool hit = !done && pb[q].key == e;
    const bool empty = !done && pb[q].key == kEncEmpty;
    r = hit ? pb[q].row : r;
    done = done || hit || empty;
  }
  if (!done) r = idmap_lookup_at(t, e, (h + kProbeBatch) & t.cap_mask, kProbeBatch);
  return r;
}

// The partition's records are read from every dedup block's
// partition-ordered copy (segment b: cnt[b] records at off[b]).  A key's
// index is the smallest place in tile order of its records: that record holds
// its first position (the records of a dedup block, and the blocks, are in
// first-position order).  Every record gets one 16-byte result at its place;
// the first records' results carry the key's count and row, in the order in
// which the first-occurrence sums and the compaction read them (a separate
// 32-byte key entry per key beside 8-byte results, which the sums and the
// compaction read again: this pass 399 us for 16.4M ids of 3.8M keys, then 331,
// the sums 70 and 33, the compaction 160 and 106; 167 / 134, 31 / 13 and 48 /
// 49 for 10.6M ids of 1.4M keys).
// A partition of at most kPartThreads * kPartFast = 2560 records is done in one
// pass with each thread's records in registers; a larger one, or one with more
// than kPartSlots = 2048 distinct keys, in sweeps of about kPartSweep records by
// a hash of the key, and if a sweep's keys do not fit (a skewed hash) the
// partition starts again with twice as many sweeps.  Where kMaxSweeps sweeps do
// not help either, rounds take as many keys as fit, so every partition ends
// with a result for each of its records.

// IDMap rows of the d keys listed in cdense; a key's row replaces it in the table.
__device__ inline void probe_keys(const TableDev& t, int d, const short* cdense, unsigned long long* ckey) {
  constexpr int NT = kPartThreads;
  constexpr int KP = 4;  // keys per thread per round: their probe batches in flight together
  for (int q0 = 0; q0 < d; q0 += KP * NT) {
    int sl[KP];
    unsigned long long e[KP];
    uint64_t h[KP];
    Slot pb[KP][kProbeBatch];
#pragma unroll
    for (int u = 0; u < KP; ++u) {
      const int q = q0 + u * NT + static_cast<int>(threadIdx.x);
      sl[u] = q < d ? cdense[q] : -1;
      e[u] = sl[u] >= 0 ? ckey[sl[u]] : kEncEmpty;
      h[u] = sl[u] >= 0 ? (idmap_hash(e[u]) & t.cap_mask) : 0;  // idle lanes read one shared line
#pragma unroll
      for (int k = 0; k < kProbeBatch; ++k) pb[u][k] = t.slots[(h[u] + k) & t.cap_mask];
    }
#pragma unroll
    for (int u = 0; u < KP; ++u)
      if (sl[u] >= 0) ckey[sl[u]] = static_cast<unsigned long long>(resolve_probe(t, e[u], h[u], pb[u]));
  }
}

// Enter key e into the LDS table (linear probing from slot h).  Returns the
// slot, or -1 if every slot holds another key.
__device__ inline int lds_insert(unsigned long long* ckey, unsigned long long e, uint64_t hh) {
  constexpr int S = kPartSlots;
  unsigned int sl = static_cast<unsigned int>(hh >> 20) & (S - 1);
  for (int probes = 0; probes < S; ++probes) {
    const unsigned long long old = atomicCAS(&ckey[sl], kEncEmpty, e);
    if (old == kEncEmpty || old == e) return static_cast<int>(sl);
    sl = (sl + 1) & (S - 1);
  }
  return -1;
}

constexpr int kRoundProbes = 64;  // probe window of a round (full windows cost as many steps per record and round)

__global__ __launch_bounds__(kPartThreads) void k_part_dedup(TableDev t, Work w) {
  constexpr int NT = kPartThreads, S = kPartSlots, OWN = S / NT, K = kPartFast;
  constexpr int kMaxSweeps = 1 << 10;
  constexpr int BPT = (kMaxDedupBlocks + NT - 1) / NT;
  __shared__ unsigned long long ckey[S];
  __shared__ unsigned int cfp[S];  // the key's index: the smallest place of its records
  __shared__ unsigned int ccnt[S];
  __shared__ short cdense[S];  // dense index -> slot
  __shared__ int cpre[kMaxDedupBlocks];   // exclusive prefix of the segment sizes
  __shared__ int cbase[kMaxDedupBlocks];  // position of each segment
  __shared__ int sh[NT / kWave + 1];
  __shared__ int ovf;
  const FrontGeom g = w.g;
  const int tid = threadIdx.x;
  // XCD-contiguous: block b runs on XCD b % 8, which takes the (b % 8)-th
  // eighth of the partitions in order, so the lines that adjacent partitions
  // share (runs of a few records per dedup block, and the count columns) are
  // fetched into one L2 (9M ids 79 -> 70 us, 16.4M 332 -> 325, 10.6M 134 -> 131)
  const int p = g.P >= 8 ? static_cast<int>(blockIdx.x % 8) * (g.P / 8) + static_cast<int>(blockIdx.x / 8)
                         : static_cast<int>(blockIdx.x);
  // the partition's segments (thread tid holds blocks tid*BPT ...)
  int cn[BPT];
  int loc = 0;
#pragma unroll
  for (int j = 0; j < BPT; ++j) {
    const int b = tid * BPT + j;
    cn[j] = b < g.nblk ? w.pcnt[static_cast<int64_t>(b) * g.P + p] : 0;
    if (b < g.nblk) cbase[b] = static_cast<int>(b * g.rcap) + w.poff[static_cast<int64_t>(b) * g.P + p];
    loc += cn[j];
  }
  int nr;
  int run = block_excl_scan<NT>(loc, sh, nr);
#pragma unroll
  for (int j = 0; j < BPT; ++j) {
    const int b = tid * BPT + j;
    if (b < g.nblk) cpre[b] = run;
    run += cn[j];
  }
  for (int q = tid; q < S; q += NT) {
    ckey[q] = kEncEmpty;
    cfp[q] = ~0u;
    ccnt[q] = 0u;
  }
  if (tid == 0) ovf = 0;
  __syncthreads();
  if (nr == 0) return;  // the whole block
  const int nb = static_cast<int>(g.nblk);
  // position of the fr-th record of the partition: the last segment whose
  // prefix is <= fr (empty segments share their successor's prefix)
  auto rec_pos = [&](int fr) {
    int lo = 0, hi = nb;  // cpre[lo] <= fr; the answer is in [lo, hi)
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (cpre[mid] <= fr) lo = mid;
      else hi = mid;
    }
    return cbase[lo] + (fr - cpre[lo]);
  };
  // dense list of the occupied slots: thread tid owns slots tid + j * NT
  // (consecutive lanes, consecutive slots: no bank conflicts), read once
  static_assert(OWN <= 32, "occupancy mask");
  auto dense_list = [&]() {
    unsigned int om = 0u;
#pragma unroll
    for (int j = 0; j < OWN; ++j) om |= static_cast<unsigned int>(ckey[j * NT + tid] != kEncEmpty) << j;
    int d;
    int at = block_excl_scan<NT>(__popc(om), sh, d);
#pragma unroll
    for (int j = 0; j < OWN; ++j)
      if ((om >> j) & 1u) cdense[at++] = static_cast<short>(j * NT + tid);
    __syncthreads();
    return d;
  };

  const bool lookup = w.kinfo != nullptr;  // else the ids partition
  // record of key `key` at place src, entered at LDS slot sl, rb occurrences
  // of its key before it (its key's row already in the table)
  auto result = [&](unsigned int src, unsigned long long key, int sl, unsigned int rb) {
    const unsigned int kidx = cfp[sl];
    const bool first = kidx == src;
    RecRes r;
    r.x = static_cast<int>(first && lookup ? ccnt[sl] : kidx);
    r.y = rb | (first ? kRecFirst : 0u);
    r.v = lookup ? static_cast<long long>(ckey[sl]) : static_cast<long long>(key ^ kSign);
    w.recres[src] = r;
  };
  bool fresh = true;  // the LDS table is clear
  if (nr <= NT * K) {
    // one pass: the thread's records tid, tid + NT, ... stay in registers (more
    // than kPartSlots distinct keys fill the table: on to the sweeps)
    int pos[K];
    TileRec x[K];
#pragma unroll
    for (int k = 0; k < K; ++k) pos[k] = tid + k * NT < nr ? rec_pos(tid + k * NT) : -1;
#pragma unroll
    for (int k = 0; k < K; ++k)
      if (pos[k] >= 0) x[k] = w.srec[pos[k]];
    int sl[K];
    unsigned int rb[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      sl[k] = -1;
      rb[k] = 0;
      if (pos[k] < 0) continue;
      sl[k] = lds_insert(ckey, x[k].key, part_hash(x[k].key));
      if (sl[k] < 0) {
        ovf = 1;
        continue;
      }
      atomicMin(&cfp[sl[k]], x[k].src);
      rb[k] = atomicAdd(&ccnt[sl[k]], x[k].meta + 1u);
    }
    __syncthreads();
    if (!ovf) {
      if (lookup) {
        const int d = dense_list();
        probe_keys(t, d, cdense, ckey);
        __syncthreads();
      }
#pragma unroll
      for (int k = 0; k < K; ++k)
        if (sl[k] >= 0) result(x[k].src, x[k].key, sl[k], rb[k]);
      return;
    }
    fresh = false;
    __syncthreads();  // every thread has read ovf before the sweeps reset it
  }

  // Rounds: ids whose hashes agree in the partition's bits and in the sweeps'
  // (they have to be made so: the hash can be inverted) do not fit any sweep.
  // A round enters keys, by another hash, until a key finds its probe window
  // full.  No slot is emptied in a round, so if one record of a key finds no
  // slot all its records find none: they wait for the next round.  Each round
  // takes at least its first record's key, so the rounds end.
  auto rounds = [&]() {
    constexpr int kToDo = -1, kDone = -2;
    for (int f = tid; f < nr; f += NT) w.ptmp[rec_pos(f)].x = kToDo;
    bool more = true;
    while (more) {
      __syncthreads();  // every thread is done with the LDS (and with ovf)
      for (int q = tid; q < S; q += NT) {
        ckey[q] = kEncEmpty;
        cfp[q] = ~0u;
        ccnt[q] = 0u;
      }
      if (tid == 0) ovf = 0;
      __syncthreads();
      for (int f = tid; f < nr; f += NT) {
        const int pos = rec_pos(f);
        if (w.ptmp[pos].x != kToDo) continue;
        const TileRec x = w.srec[pos];
        unsigned int sl = static_cast<unsigned int>(idmap_hash(x.key) >> 20) & (S - 1);
        bool in = false;
#pragma unroll 1
        for (int probes = 0; probes < kRoundProbes && !in; ++probes) {
          const unsigned long long old = atomicCAS(&ckey[sl], kEncEmpty, x.key);
          in = old == kEncEmpty || old == x.key;
          if (!in) sl = (sl + 1) & (S - 1);
        }
        if (!in) {
          ovf = 1;
          continue;
        }
        atomicMin(&cfp[sl], x.src);
        w.ptmp[pos] = make_int2(static_cast<int>(sl), static_cast<int>(atomicAdd(&ccnt[sl], x.meta + 1u)));
      }
      __syncthreads();
      more = ovf != 0;
      for (int f = tid; f < nr; f += NT) {
        const int pos = rec_pos(f);
        const int2 tp = w.ptmp[pos];
        if (tp.x < 0) continue;
        const TileRec x = w.srec[pos];
        if (lookup && cfp[tp.x] == x.src)  // the key's first record alone carries its row
          ckey[tp.x] = static_cast<unsigned long long>(idmap_lookup(t, x.key));
        result(x.src, x.key, tp.x, static_cast<unsigned int>(tp.y));
        w.ptmp[pos].x = kDone;
      }
    }
  };

  // sweeps: a partition above the register pass (ids that hardly repeat, or a
  // skewed hash).  Sweep s takes the keys whose 20 hash bits mod nsw are s (a
  // 32-bit remainder).  KS records per thread and round: their loads are in
  // flight together.
  constexpr int KS = 4;
  int nsw = min((nr + kPartSweep - 1) / kPartSweep, kMaxSweeps);
  auto sweep_of = [&](uint64_t h) {
    return static_cast<int>((static_cast<uint32_t>(h) & 0xFFFFFu) % static_cast<uint32_t>(nsw));
  };
  int s = 0;
  while (s < nsw) {
    if (!fresh) {
      for (int q = tid; q < S; q += NT) {
        ckey[q] = kEncEmpty;
        cfp[q] = ~0u;
        ccnt[q] = 0u;
      }
    }
    fresh = false;
    if (tid == 0) ovf = 0;
    __syncthreads();
    for (int f0 = tid; f0 < nr; f0 += KS * NT) {
      int pos[KS];
      TileRec x[KS];
#pragma unroll
      for (int k = 0; k < KS; ++k) {
        pos[k] = f0 + k * NT < nr ? rec_pos(f0 + k * NT) : -1;
        if (pos[k] >= 0) x[k] = w.srec[pos[k]];
      }
#pragma unroll
      for (int k = 0; k < KS; ++k) {
        if (pos[k] < 0) continue;
        const uint64_t h = part_hash(x[k].key);
        if (sweep_of(h) != s) continue;
        const int sl = lds_insert(ckey, x[k].key, h);
        if (sl < 0) {
          ovf = 1;
          continue;
        }
        atomicMin(&cfp[sl], x[k].src);
        const unsigned int rb = atomicAdd(&ccnt[sl], x[k].meta + 1u);
        w.ptmp[pos[k]] = make_int2(sl, static_cast<int>(rb));
      }
    }
    __syncthreads();
    if (ovf) {
      __syncthreads();  // every thread has read ovf
      if (__builtin_expect(nsw >= kMaxSweeps, 0)) {
        rounds();
        return;
      }
      nsw *= 2;
      s = 0;
      continue;
    }
    if (lookup) {
      const int d = dense_list();
      probe_keys(t, d, cdense, ckey);
      __syncthreads();
    }
    for (int f0 = tid; f0 < nr; f0 += KS * NT) {
      int pos[KS];
      TileRec x[KS];
      int2 tp[KS];
#pragma unroll
      for (int k = 0; k < KS; ++k) {
        pos[k] = f0 + k * NT < nr ? rec_pos(f0 + k * NT) : -1;
        if (pos[k] >= 0) {
          x[k] = w.srec[pos[k]];
          tp[k] = w.ptmp[pos[k]];  // unset, or another sweep's, where the record is another sweep's
        }
      }
#pragma unroll
      for (int k = 0; k < KS; ++k)
        if (pos[k] >= 0 && sweep_of(part_hash(x[k].key)) == s)
          result(x[k].src, x[k].key, tp[k].x, static_cast<unsigned int>(tp[k].y));
    }
    ++s;
    __syncthreads();  // the next sweep clears the LDS
  }
}

// ---------------------------------------------------------------------------
// pass 5: tile sums over the first occurrences
// ---------------------------------------------------------------------------

__device__ inline void load4(const int32_t* __restrict__ p, int64_t i0, int64_t n, int (&v)[4]) {
  if (i0 + 4 <= n) {
    const int4 a = *reinterpret_cast<const int4*>(p + i0);
    v[0] = a.x;
    v[1] = a.y;
    v[2] = a.z;
    v[3] = a.w;
  } else {
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = (i0 + k < n) ? p[i0 + k] : -1;
  }
}

// Record tile rt: its dedup block, and the place of its first record slot.
struct RecTile {
  uint32_t blk, at, left;  // left: records of the dedup block from `at` on (<= 0 as a signed number: none)
};

__device__ inline RecTile rec_tile(const Work& w, uint32_t rt) {
  const uint32_t per = static_cast<uint32_t>(w.g.rcap / kRankTile);  // record tiles per dedup block
  RecTile x;
  x.blk = rt / per;  // 32 bits: places are below 2^28
  const uint32_t r0 = (rt - x.blk * per) * kRankTile;
  x.at = x.blk * static_cast<uint32_t>(w.g.rcap) + r0;
  x.left = static_cast<uint32_t>(w.nrec[x.blk]) - r0;
  return x;
}

// The tile lies wholly past its dedup block's records (a block's record slots
// are sized for its ids, and distinct keys are fewer).
__device__ inline bool empty_tile(const RecTile& x) { return static_cast<int32_t>(x.left) <= 0; }

// The results of 4 record slots per thread (a key's first record is its only
// one that is counted); first[k]: slot k holds a first record.
__device__ inline void load_results(const Work& w, const RecTile& x, RecRes (&r)[4], bool (&first)[4]) {
#pragma unroll
  for (int k = 0; k < 4; ++k) r[k] = w.recres[x.at + threadIdx.x * 4 + k];
#pragma unroll
  for (int k = 0; k < 4; ++k)
    first[k] = static_cast<int32_t>(threadIdx.x * 4 + k) < static_cast<int32_t>(x.left) && (r[k].y & kRecFirst);
}

// What a tile's four slots of a thread add to the sums: keys, their counts,
// keys not found, hot keys, hot-key units.
__device__ inline void sum_firsts(const RecRes (&r)[4], const bool (&first)[4], int maxu, int (&v)[5]) {
#pragma unroll
  for (int a = 0; a < 5; ++a) v[a] = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (!first[k]) continue;
    v[0] += 1;
    v[1] += r[k].x;
    v[2] += r[k].v < 0;
    if (r[k].x > kLong) {
      v[3] += 1;
      v[4] += unit_count(r[k].x, maxu);
    }
  }
}

// Per record tile: sums over its first records.  Record tiles in block-major
// order list the keys in the order of their first positions.
template <int NT>
__global__ __launch_bounds__(NT) void k_first_sums(Work w) {
  __shared__ int sh[NT / kWave][5];
  const RecTile x = rec_tile(w, blockIdx.x);
  if (empty_tile(x)) {  // block-uniform
    if (threadIdx.x < 5) w.bsum[threadIdx.x * w.ntiles + blockIdx.x] = 0;
    return;
  }
  RecRes r[4];
  bool first[4];
  load_results(w, x, r, first);
  int v[5];
  sum_firsts(r, first, w.maxu, v);
#pragma unroll
  for (int a = 0; a < 5; ++a) v[a] = wave_sum(v[a]);
  if ((threadIdx.x & (kWave - 1)) == 0) {
#pragma unroll
    for (int a = 0; a < 5; ++a) sh[threadIdx.x / kWave][a] = v[a];
  }
  __syncthreads();
  if (threadIdx.x < 5) {
    int tot = 0;
#pragma unroll
    for (int q = 0; q < NT / kWave; ++q) tot += sh[q][threadIdx.x];
    w.bsum[threadIdx.x * w.ntiles + blockIdx.x] = tot;
  }
}

// ---------------------------------------------------------------------------
// one-block scan of the five tile-sum arrays; row reservation
// ---------------------------------------------------------------------------

__device__ inline void publish_live(int64_t* h_live, int64_t tag, int64_t live) {
  // one 8-byte store to pinned host memory: (call tag << 48) | live rows
  if (h_live) {
    *reinterpret_cast<volatile int64_t*>(h_live) = (tag << 48) | live;
    __threadfence_system();
  }
}

// Rows for `req` keys not found, from `hw` rows allocated, `keys` live keys
// and `F` free rows: as many as both the IDMap (its key limit counts the
// tombstones) and the Blocks (free rows, then provisioned ones) allow.  The
// first min(inserted, F) new keys take free rows.  The published count
// bounds both the IDMap occupancy and the rows allocated.
struct Reservation {
  int64_t ins, hw, ftop, take;  // inserted, rows allocated and free rows before, free rows taken
  int64_t published;            // the live count's bound after the call
};

// tcap: {key limit, provisioned rows, tombstones} of the table
__device__ inline Reservation reservation(int64_t req, int64_t hw, int64_t keys, int64_t F, const int64_t (&tcap)[3]) {
  const int64_t tombs = tcap[2];
  const int64_t key_room = max(tcap[0] - keys - tombs, int64_t(0));
  const int64_t row_room = F + max(tcap[1] - hw, int64_t(0));
  const int64_t ins = min(req, min(key_room, row_room));
  const int64_t take = min(ins, F);
  return Reservation{ins, hw, F, take, max(keys + ins + tombs, hw + ins - take)};
}

__device__ inline void store_reservation(int64_t* cscal, int64_t* tscal, int64_t req, int64_t keys,
                                         const Reservation& r) {
  cscal[kCNew] = r.ins;
  cscal[kCBaseLive] = r.hw;
  cscal[kCBaseKeys] = keys;
  cscal[kCFreeTop] = r.ftop;
  cscal[kCFreeTake] = r.take;
  cscal[kCTrunc] = req > r.ins ? 1 : 0;
  tscal[kTLive] = r.hw + r.ins - r.take;
  tscal[kTKeys] = keys + r.ins;
  tscal[kTFree] = r.ftop - r.take;
}

// Scan of the five tile-sum arrays: block c scans chunk c (kScanChunk tiles,
// R per thread) in place and stores the chunk's totals; the last block to
// finish (a counter, no waiting) scans the chunk totals in place and reserves
// the rows of the new keys.  A tile's prefix is then bsum[a][tile] + csum[a][tile / kScanChunk].
template <int R>
__global__ __launch_bounds__(1024) void k_scan5(int32_t* __restrict__ bsum, int64_t nb, int64_t ntiles,
                                                int32_t* __restrict__ csum, int64_t nch, int64_t* cscal,
                                                int64_t* tscal) {
  static_assert(1024 * R == kScanChunk, "one chunk per block");
  __shared__ int sh[1024 / kWave + 1][5];
  __shared__ bool last;
  const int64_t c = blockIdx.x;
  const int64_t lo = c * kScanChunk + static_cast<int64_t>(threadIdx.x) * R;
  int64_t ts[6];  // the table's scalars, read ahead of the scan (the last block's first thread uses them)
#pragma unroll
  for (int q = 0; q < 6; ++q) ts[q] = tscal[q == 5 ? kTTomb : q == 4 ? kTFree : q == 3 ? kTKeys : q == 2 ? kTRowCap : q];
  int v[5][R];
#pragma unroll
  for (int a = 0; a < 5; ++a)
#pragma unroll
    for (int j = 0; j < R; ++j) v[a][j] = lo + j < nb ? bsum[a * ntiles + lo + j] : 0;
  int local[5], ex[5], tot[5];
#pragma unroll
  for (int a = 0; a < 5; ++a) {
    local[a] = 0;
#pragma unroll
    for (int j = 0; j < R; ++j) local[a] += v[a][j];
  }
  block_excl_scan5<1024>(local, ex, tot, sh);
#pragma unroll
  for (int a = 0; a < 5; ++a) {
    int run = ex[a];
#pragma unroll
    for (int j = 0; j < R; ++j) {
      if (lo + j < nb) bsum[a * ntiles + lo + j] = run;
      run += v[a][j];
    }
  }
  if (nch == 1) {
    // one chunk: its totals are the totals (no chunk scan, no counter)
    if (threadIdx.x < 5) csum[threadIdx.x] = 0;
  } else {
    if (threadIdx.x == 0) {
#pragma unroll
      for (int a = 0; a < 5; ++a) csum[a * nch + c] = tot[a];
      __threadfence();
      const unsigned long long done =
          atomicAdd(reinterpret_cast<unsigned long long*>(&cscal[kCScanDone]), 1ull);
      last = done == static_cast<unsigned long long>(nch - 1);
    }
    __syncthreads();
    if (!last) return;
    __threadfence();
    // the last block: exclusive scan of the chunk totals (nch <= 1024 R)
    int cv[5][R];
    const int64_t clo = static_cast<int64_t>(threadIdx.x) * R;
#pragma unroll
    for (int a = 0; a < 5; ++a)
#pragma unroll
      for (int j = 0; j < R; ++j)
        cv[a][j] = clo + j < nch ? __hip_atomic_load(&csum[a * nch + clo + j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
#pragma unroll
    for (int a = 0; a < 5; ++a) {
      local[a] = 0;
#pragma unroll
      for (int j = 0; j < R; ++j) local[a] += cv[a][j];
    }
    block_excl_scan5<1024>(local, ex, tot, sh);
#pragma unroll
    for (int a = 0; a < 5; ++a) {
      int run = ex[a];
#pragma unroll
      for (int j = 0; j < R; ++j) {
        if (clo + j < nch) csum[a * nch + clo + j] = run;
        run += cv[a][j];
      }
    }
  }
  if (threadIdx.x != 0) return;
  cscal[kCScanDone] = 0;  // ready for the next call on this workspace
  cscal[kCU] = tot[0];
  cscal[kCValid] = tot[1];
  cscal[kCNewReq] = tot[2];
  cscal[kCNLong] = tot[3];
  cscal[kCNUnits] = tot[4];
  const int64_t tcap[3] = {ts[1], ts[2], ts[5]};
  const Reservation r = reservation(tot[2], ts[0], ts[3], ts[4], tcap);
  store_reservation(cscal, tscal, tot[2], ts[3], r);
}

// After the host grew the table: reserve again from the same counts.
__global__ void k_rereserve(int64_t* cscal, int64_t* tscal) {
  const int64_t tcap[3] = {tscal[kTLimit], tscal[kTRowCap], tscal[kTTomb]};
  const Reservation r = reservation(cscal[kCNewReq], cscal[kCBaseLive], cscal[kCBaseKeys], cscal[kCFreeTop], tcap);
  store_reservation(cscal, tscal, cscal[kCNewReq], cscal[kCBaseKeys], r);
}

__global__ void k_zero_scalars(int64_t* cscal) { cscal[threadIdx.x] = 0; }

hipError_t launch_rereserve(const Work& w, const TableDev& t, hipStream_t s) {
  k_rereserve<<<1, 1, 0, s>>>(w.scal, t.scal);
  return hipGetLastError();
}

FrontGeom front_geom(int64_t n) {
  FrontGeom g;
  const int64_t n1 = n > 0 ? n : 1;
  g.ntiles = (n1 + kDedupTile - 1) / kDedupTile;
  g.R = std::min<int64_t>(kMaxTilesPerBlock, (g.ntiles + 255) / 256);
  g.nblk = (g.ntiles + g.R - 1) / g.R;
  g.rcap = g.R * kDedupTile;
  g.P = 1;
  g.logP = 0;
  // about 4096 ids (some 1500-2000 records) per partition: the partitions of
  // a batch up to ~3M ids are all resident at once (3 blocks per CU by their
  // registers; their 40 KB of LDS would admit four)
  while (g.P < kMaxParts && static_cast<int64_t>(g.P) * 4096 < n1) {
    g.P <<= 1;
    ++g.logP;
  }
  return g;
}

hipError_t launch_dedup_keys(const int64_t* values, int64_t n, const TableDev& t, const Work& w, hipEvent_t* ev_tile,
                             hipEvent_t* ev_part, hipStream_t s) {
  const FrontGeom& g = w.g;
  if (n <= 0 || g.nblk > kMaxDedupBlocks) return hipErrorInvalidValue;
  if (ev_tile && ev_tile[0]) (void)hipEventRecord(ev_tile[0], s);
  k_tile_dedup<kDedupThreads><<<static_cast<unsigned>(g.nblk), kDedupThreads, 0, s>>>(
      values, n, w, reinterpret_cast<int*>(t.scal + kTErr));
  if (ev_tile && ev_tile[1]) (void)hipEventRecord(ev_tile[1], s);
  if (ev_part && ev_part[0]) (void)hipEventRecord(ev_part[0], s);
  k_part_dedup<<<static_cast<unsigned>(g.P), kPartThreads, 0, s>>>(t, w);
  return hipGetLastError();
}

hipError_t launch_dedup_probe(const int64_t* values, int64_t n, const TableDev& t, const Work& w, hipEvent_t* ev_tile,
                              hipEvent_t* ev_part, hipStream_t s) {
  if (n <= 0) {
    k_zero_scalars<<<1, kCScalars, 0, s>>>(w.scal);
    return hipGetLastError();
  }
  const hipError_t e = launch_dedup_keys(values, n, t, w, ev_tile, ev_part, s);
  if (e != hipSuccess) return e;
  const int64_t nb = record_tiles(w.g);
  k_first_sums<kBlock><<<static_cast<unsigned>(nb), kBlock, 0, s>>>(w);
  const int64_t nch = (nb + kScanChunk - 1) / kScanChunk;
  k_scan5<kScanChunk / 1024><<<static_cast<unsigned>(nch), 1024, 0, s>>>(w.bsum, nb, w.ntiles, w.csum, nch, w.scal,
                                                                          t.scal);
  if (ev_part && ev_part[1]) (void)hipEventRecord(ev_part[1], s);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// pass 7: unique ids, segments, rows, IDMap inserts
// ---------------------------------------------------------------------------

template <int NT>
__global__ __launch_bounds__(NT) void k_compact(TableDev t, Work w, int64_t* h_live, int64_t tag) {
  __shared__ int sh[NT / kWave + 1][5];
  const int b = blockIdx.x;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    if (w.scal[kCTrunc]) atomicOr(reinterpret_cast<int*>(&t.scal[kTErr]), kErrFull);
    // the host's bound on the live count, published here and not at the end of
    // the scan: a store to host memory that no launch waits for behind it
    publish_live(h_live, tag, max(t.scal[kTKeys] + t.scal[kTTomb], t.scal[kTLive]));
  }
  const RecTile x = rec_tile(w, b);
  if (empty_tile(x)) return;  // block-uniform: no keys, nothing to write
  int pre[5];  // the record tile's exclusive prefixes (keys, count, new, hot, units)
  const int64_t nch = (static_cast<int64_t>(gridDim.x) + kScanChunk - 1) / kScanChunk;
#pragma unroll
  for (int a = 0; a < 5; ++a) pre[a] = w.bsum[a * w.ntiles + b] + w.csum[a * nch + b / kScanChunk];
  RecRes r[4];
  bool first[4];
  load_results(w, x, r, first);
  unsigned long long ek[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) ek[k] = w.trec[x.at + threadIdx.x * 4 + k].key;  // all reads in flight together
  // the tile's keys get consecutive unique ids, segments, rows of new keys,
  // hot-key indices and backward units
  int v[5], ex[5], tot[5];
  sum_firsts(r, first, w.maxu, v);
  block_excl_scan5<NT>(v, ex, tot, sh);
  int uid = pre[0] + ex[0];
  int start = pre[1] + ex[1];
  int64_t nr = pre[2] + ex[2];
  int lnext = pre[3] + ex[3];
  int unext = pre[4] + ex[4];
  const int64_t inserted = w.scal[kCNew];
  const int64_t live0 = w.scal[kCBaseLive];
  const int64_t ftop = w.scal[kCFreeTop], ftake = w.scal[kCFreeTake];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (!first[k]) continue;
    const int c = r[k].x;
    const int64_t key = static_cast<int64_t>(ek[k] ^ kSign);
    w.unique[uid] = key;
    if (c > kLong) {
      w.long_u[lnext] = uid;
      w.long_start[lnext] = unext;
      ++lnext;
      unext += unit_count(c, w.maxu);
    }
    int64_t row = r[k].v;
    if (row < 0) {
      if (nr < inserted) {
        const int64_t slot = idmap_claim(t, ek[k]);
        if (slot >= 0) {
          // the first `ftake` new keys take free rows from the top of the stack
          row = nr < ftake ? t.free_rows[ftop - 1 - nr] : live0 + (nr - ftake);
          t.slots[slot].row = row;
          w.new_list[nr] = uid;
        } else {
          w.new_list[nr] = -1;  // no slot (cannot happen below the key limit): no row to initialise
          atomicOr(reinterpret_cast<int*>(&t.scal[kTErr]), kErrProbe);
        }
      }
      ++nr;
    } else if (t.meta_off >= 0) {
      // eviction: this call is the key's last lookup
      *reinterpret_cast<uint32_t*>(t.store.row(row) + t.meta_off + 8) = t.clock;
    }
    w.rows[uid] = row;
    w.useg[uid] = Seg{row, start, c};
    w.kinfo[x.at + threadIdx.x * 4 + k] = KeyInfo{row, uid, start};
    ++uid;
    start += c;
  }
}

// The initial value of element j of a new key's row: 24 bits of the
// (j+1)-th splitmix64 output from state mix(key ^ mix(seed)), mapped
// exactly onto [0, 1), then one fp32 fused multiply-add onto [lo, hi].
__device__ inline float init_value(uint64_t z, int j, float lo, float span) {
  const uint64_t h = mix64(z + static_cast<uint64_t>(j + 1) * 0x9E3779B97F4A7C15ull);
  const float u = static_cast<float>(h >> 40) * 0x1.0p-24f;
  return __builtin_fmaf(u, span, lo);
}

// A lane group of 16 (lane = 0 ... 15) writes a new key's row: w from the init
// formula, optimizer state zero, and for eviction the key and this call's
// clock; 16 bytes per lane per store.
constexpr int kInitLanes = 16;

__device__ inline void init_row(const TableDev& t, int64_t row, int64_t key, int lane) {
  const int chunks = static_cast<int>(t.store.stride / 16);
  const int wbytes = t.dim * (t.row_dtype ? 2 : 4);
  const uint64_t z = mix64(static_cast<uint64_t>(key) ^ mix64(t.seed));
  uint8_t* rp = t.store.row(row);
  for (int ch = lane; ch < chunks; ch += kInitLanes) {
    const int off = ch * 16;
    uint4 val = make_uint4(0u, 0u, 0u, 0u);
    if (off < wbytes) {
      if (t.row_dtype == 0) {
        const int j0 = off / 4;
        val = make_uint4(__float_as_uint(init_value(z, j0, t.lo, t.span)),
                         __float_as_uint(init_value(z, j0 + 1, t.lo, t.span)),
                         __float_as_uint(init_value(z, j0 + 2, t.lo, t.span)),
                         __float_as_uint(init_value(z, j0 + 3, t.lo, t.span)));
      } else {
        const int j0 = off / 2;
        uint32_t h[4];
#pragma unroll
        for (int k = 0; k < 4; ++k)
          h[k] = static_cast<uint32_t>(f32_to_bf16(init_value(z, j0 + 2 * k, t.lo, t.span))) |
                 (static_cast<uint32_t>(f32_to_bf16(init_value(z, j0 + 2 * k + 1, t.lo, t.span))) << 16);
        val = make_uint4(h[0], h[1], h[2], h[3]);
      }
    }
    if (t.meta_off >= 0 && off + 16 > t.meta_off && off < t.meta_off + 12) {
      uint32_t v4[4] = {val.x, val.y, val.z, val.w};
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const int b = off + 4 * q4 - t.meta_off;  // byte of the {key, clock} record
        if (b == 0) v4[q4] = static_cast<uint32_t>(static_cast<uint64_t>(key));
        if (b == 4) v4[q4] = static_cast<uint32_t>(static_cast<uint64_t>(key) >> 32);
        if (b == 8) v4[q4] = t.clock;
      }
      val = make_uint4(v4[0], v4[1], v4[2], v4[3]);
    }
    *reinterpret_cast<uint4*>(rp + off) = val;
  }
}

// The rows of the inserted keys: block `blk` of `nblk` takes every nblk-th
// group of keys.
__device__ inline void init_rows(const TableDev& t, const Work& w, int64_t blk, int64_t nblk) {
  constexpr int G = kInitLanes;
  const int64_t inserted = w.scal[kCNew];
  for (int64_t q = blk * (kBlock / G) + threadIdx.x / G; q < inserted; q += nblk * (kBlock / G)) {
    const int u = w.new_list[q];
    if (u >= 0) init_row(t, w.useg[u].row, w.unique[u], threadIdx.x % G);
  }
}

// The per-occurrence pass: inverse[i] = unique id of occurrence i (-1 for a
// rejected key).  For a forward (OCC) it also writes each occurrence's row
// and its position in the occurrence list (the key's segment start + the
// occurrences of the key before the record + the rank inside the tile).
template <bool OCC>
__device__ inline void occ_pass(const Work& w, int64_t n, uint32_t blk) {
  const int64_t i0 = (static_cast<int64_t>(blk) * kBlock + threadIdx.x) * 4;
  if (i0 >= n) return;
  // a block's kBlock * 4 ids lie in one dedup tile: its records' place is the same for all
  static_assert(kDedupTile % (kBlock * 4) == 0, "a block's ids share a dedup tile");
  const uint32_t tile = blk / (kDedupTile / (kBlock * 4));
  const uint32_t base = tile / static_cast<uint32_t>(w.g.R) * static_cast<uint32_t>(w.g.rcap);
  int ow[4];
  load4(reinterpret_cast<const int32_t*>(w.occ_word), i0, n, ow);  // -1 = kOccRejected past n
  uint2 rr[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint32_t o = static_cast<uint32_t>(ow[k]);
    rr[k] = *reinterpret_cast<const uint2*>(&w.recres[o == kOccRejected ? 0u : base + (o >> 12)]);  // x, y: all in flight together
  }
  KeyInfo a[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint32_t o = static_cast<uint32_t>(ow[k]);
    const uint32_t kidx = rr[k].y & kRecFirst ? base + (o >> 12) : rr[k].x;
    // (clamped: no result could become a wild read)
    a[k] = w.kinfo[o == kOccRejected ? 0u : min(kidx, static_cast<uint32_t>(w.nkeyidx - 1))];
  }
  int pos[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint32_t o = static_cast<uint32_t>(ow[k]);
    pos[k] = a[k].start + static_cast<int>(rr[k].y & ~kRecFirst) + static_cast<int>(o & 0xFFFu);
    if (o == kOccRejected) {
      a[k].row = -1;
      a[k].uid = -1;
      pos[k] = -1;
    }
  }
  if (i0 + 4 <= n) {
    // the inverse (the caller's) and the list positions (the backward's)
    // are not read in the forward: non-temporal
    store4_nt(w.inverse + i0, a[0].uid, a[1].uid, a[2].uid, a[3].uid);
    if (OCC) {
      *reinterpret_cast<longlong2*>(w.occ_row + i0) = make_longlong2(a[0].row, a[1].row);
      *reinterpret_cast<longlong2*>(w.occ_row + i0 + 2) = make_longlong2(a[2].row, a[3].row);
      if (w.list) {  // the pool reads the positions next, and fills the list: no gradient row yet
        *reinterpret_cast<int4*>(w.occ_pos + i0) = make_int4(pos[0], pos[1], pos[2], pos[3]);
        *reinterpret_cast<int4*>(w.occ_ref + i0) = make_int4(-1, -1, -1, -1);
      } else {
        store4_nt(w.occ_pos + i0, pos[0], pos[1], pos[2], pos[3]);
      }
    }
  } else {
    for (int k = 0; k < 4 && i0 + k < n; ++k) {
      w.inverse[i0 + k] = a[k].uid;
      if (OCC) {
        w.occ_row[i0 + k] = a[k].row;
        w.occ_pos[i0 + k] = pos[k];
        if (w.list) w.occ_ref[i0 + k] = -1;
      }
    }
  }
}

// Backward units of the hot keys, one per thread: the hot key of unit y is the
// last one whose first unit is <= y.
__device__ inline void write_unit(const Work& w, int64_t y) {
  if (y >= w.scal[kCNUnits]) return;
  int lo = 0, hi = static_cast<int>(w.scal[kCNLong]);
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (w.long_start[mid] <= y) lo = mid;
    else hi = mid;
  }
  const Seg sg = w.useg[w.long_u[lo]];
  const int usz = kUnit << unit_shift(sg.count, w.maxu), j = static_cast<int>(y) - w.long_start[lo];
  w.units[y] = Unit{lo, sg.start + j * usz, sg.start + min((j + 1) * usz, sg.count), 0};
}

// The last pass of a lookup: blocks [0, occ_blocks) run the per-occurrence
// pass, the next unit_blocks write the hot keys' units, the others the rows of
// the inserted keys (all only need the compaction, so they share one launch).
template <bool OCC>
__global__ __launch_bounds__(kBlock) void k_occ_init(TableDev t, Work w, int64_t n, uint32_t occ_blocks,
                                                     uint32_t unit_blocks) {
  const uint32_t b = blockIdx.x;
  // the blocks of a dedup tile on one XCD: they read the same records' results
  if (b < occ_blocks) occ_pass<OCC>(w, n, xcd_runs<kDedupTile / (kBlock * 4)>(b, occ_blocks));
  else if (b - occ_blocks < unit_blocks) write_unit(w, static_cast<int64_t>(b - occ_blocks) * kBlock + threadIdx.x);
  else init_rows(t, w, b - occ_blocks - unit_blocks, gridDim.x - occ_blocks - unit_blocks);
}

hipError_t launch_compact_insert(int64_t n, const TableDev& t, const Work& w, bool occ_lists, int64_t* h_live,
                                 int64_t tag, hipEvent_t* ev_compact, hipEvent_t* ev_init, hipEvent_t* ev_occ,
                                 hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int64_t nb = record_tiles(w.g);
  if (ev_compact && ev_compact[0]) (void)hipEventRecord(ev_compact[0], s);
  k_compact<kBlock><<<static_cast<unsigned>(nb), kBlock, 0, s>>>(t, w, h_live, tag);
  if (ev_compact && ev_compact[1]) (void)hipEventRecord(ev_compact[1], s);
  // one launch: the per-occurrence pass and the new rows (the init-rows and
  // occurrence events both bracket it)
  if (ev_init && ev_init[0]) (void)hipEventRecord(ev_init[0], s);
  if (ev_occ && ev_occ[0]) (void)hipEventRecord(ev_occ[0], s);
  const unsigned ob = grid_for(n, kBlock * 4, 1ll << 31);
  const unsigned ib = grid_for(n, kBlock / 16, 8192);
  const unsigned ub = occ_lists ? grid_for(2 * (n / kUnit) + 2, kBlock) : 0u;
  if (occ_lists) k_occ_init<true><<<static_cast<unsigned>(ob + ub + ib), kBlock, 0, s>>>(t, w, n, ob, ub);
  else k_occ_init<false><<<static_cast<unsigned>(ob + ib), kBlock, 0, s>>>(t, w, n, ob, 0u);
  if (ev_occ && ev_occ[1]) (void)hipEventRecord(ev_occ[1], s);
  if (ev_init && ev_init[1]) (void)hipEventRecord(ev_init[1], s);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// a small batch: the front end in two launches
// ---------------------------------------------------------------------------
//
// At most kSmallIds ids: every launch of the general front end is a chain of
// dependent memory trips of 4-12 us here (46 us for 4750 ids; two partitions
// of 3300 distinct ids each even fall into the sweeps: 123 us for 6656 ids).
//   k_small_dedup  block b takes the ids of hash partition b: LDS dedup and
//                  the IDMap probe of each key, results by position
//   k_small_rows   every block scans the counts of all positions (unique ids,
//                  segments, new keys); the ids are split over the blocks,
//                  which insert, write the new rows and every result
// Several blocks because one CU has too few misses in flight for the probes
// (7 us for 4096 keys) and issues the per-id work too slowly: the same front
// end in one block plus a launch for the new rows took 23 us for 4750 ids and
// 31 us for 6656, these two 14.7 and 15.5 us.
// Any split of the keys over the blocks fits: the LDS arrays hold the whole
// batch.

constexpr int kSmallNT = 1024;
constexpr int kSmallPT = kSmallIds / kSmallNT;  // positions per thread
constexpr int kSmallPart = 512;                  // ids per block, about
constexpr uint32_t kSmallNew = 0x80000000u;      // in a count: the key was not found

// The partition of an encoded key (2^logG partitions).
__device__ inline uint32_t small_part(unsigned long long e, int logG) {
  const uint32_t x = (static_cast<uint32_t>(e) ^ static_cast<uint32_t>(e >> 32) * 0x9E3779B1u) * 0x85EBCA6Bu;
  return logG == 0 ? 0u : (x ^ (x >> 15)) * 0xC2B2AE35u >> (32 - logG);
}

// What the two launches hand over beside the results' own arrays, in arrays of
// the general passes: the counts by position, the table's scalars as they were
// before the call (the second launch changes them).
__device__ inline uint32_t* small_counts(const Work& w) { return reinterpret_cast<uint32_t*>(w.ptmp); }
__device__ inline int64_t* small_scalars(const Work& w) { return reinterpret_cast<int64_t*>(w.bsum); }
static_assert(kTScalars * sizeof(int64_t) <= 5 * (kDedupTile / kRankTile) * sizeof(int32_t),
              "the smallest tile-sum array holds the table's scalars");

// Per id i of the block's partition: occ_word = first position of its key << 16
// | rank among the key's ids (kOccRejected for a reserved key), and its count:
// at a first position the key's count | kSmallNew if it was not found (and
// occ_row = its row), 0 elsewhere.
__global__ __launch_bounds__(kSmallNT) void k_small_dedup(const int64_t* __restrict__ values, int n, int logG, TableDev t,
                                                          Work w) {
  constexpr int NT = kSmallNT, PT = kSmallPT;
  constexpr unsigned int kNone = 0xFFFFFFFFu;
  constexpr int kIdx = 13;  // bits of a member index
  static_assert(kSmallIds <= 1 << kIdx, "slot = first position << kIdx | member, below kNone");
  __shared__ unsigned long long lkey[kSmallIds];           // the members' keys
  __shared__ alignas(16) unsigned int slot[kSmallIds];     // LDS hash: smallest (position, member) of the slot's key
  __shared__ alignas(16) unsigned int cnt2[kSmallIds / 2]; // occurrences by first member, 16 bits each
  __shared__ unsigned short lpos[kSmallIds], lslot[kSmallIds];
  __shared__ int members;
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  unsigned long long e[PT];
#pragma unroll
  for (int k = 0; k < PT; ++k)  // clamped, not skipped: all in flight together
    e[k] = static_cast<unsigned long long>(values[min(k * NT + tid, n - 1)]) ^ kSign;
  if (tid == 0) members = 0;
  for (int q = tid; q < kSmallIds / 4; q += NT) reinterpret_cast<uint4*>(slot)[q] = make_uint4(kNone, kNone, kNone, kNone);
  for (int q = tid; q < kSmallIds / 8; q += NT) reinterpret_cast<uint4*>(cnt2)[q] = make_uint4(0u, 0u, 0u, 0u);
  if (blockIdx.x == 0 && tid < kTScalars) small_scalars(w)[tid] = t.scal[tid];
  __syncthreads();
  const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll
  for (int k = 0; k < PT; ++k) {
    if (k * NT >= n) continue;  // block-uniform
    const int i = k * NT + tid;
    bool mine = i < n && small_part(e[k], logG) == blockIdx.x;
    if (mine && e[k] <= kEncTomb) {
      atomicOr(reinterpret_cast<int*>(&t.scal[kTErr]), kErrKey);
      w.occ_word[i] = kOccRejected;
      small_counts(w)[i] = 0u;
      mine = false;
    }
    const uint64_t b = __ballot(mine);
    int at = 0;
    if (lane == 0 && b) at = atomicAdd(&members, __popcll(b));
    at = __shfl(at, 0, kWave) + __popcll(b & below);
    if (mine) {
      lkey[at] = e[k];
      lpos[at] = static_cast<unsigned short>(i);
    }
  }
  __syncthreads();
  const int M = members;
  for (int m = tid; m < M; m += NT) {
    const unsigned long long key = lkey[m];
    const unsigned int x = static_cast<unsigned int>(lpos[m]) << kIdx | static_cast<unsigned int>(m);
    unsigned int sl = static_cast<unsigned int>(idmap_hash(key) >> 40) & (kSmallIds - 1);
    while (true) {  // at most as many keys as slots: terminates
      const unsigned int old = atomicCAS(&slot[sl], kNone, x);
      if (old == kNone) break;
      if (lkey[old & (kSmallIds - 1)] == key) {  // a slot only ever changes to a smaller position of its key
        if (x < old) atomicMin(&slot[sl], x);
        break;
      }
      sl = (sl + 1) & (kSmallIds - 1);
    }
    lslot[m] = static_cast<unsigned short>(sl);
  }
  __syncthreads();
  for (int m = tid; m < M; m += NT) {
    const unsigned int f = slot[lslot[m]];
    const int fm = static_cast<int>(f & (kSmallIds - 1)), sft = (fm & 1) * 16;
    const unsigned int rank = (atomicAdd(&cnt2[fm >> 1], 1u << sft) >> sft) & 0xFFFFu;
    w.occ_word[lpos[m]] = (f >> kIdx) << 16 | rank;
  }
  __syncthreads();
  for (int m = tid; m < M; m += NT) {
    const int i = lpos[m];
    uint32_t c = 0u;
    if (static_cast<int>(slot[lslot[m]] & (kSmallIds - 1)) == m) {
      const int64_t r = idmap_lookup(t, lkey[m]);
      c = (cnt2[m >> 1] >> ((m & 1) * 16)) & 0xFFFFu;
      if (r < 0) c |= kSmallNew;
      w.occ_row[i] = r;
    }
    small_counts(w)[i] = c;
  }
}

template <bool OCC>
__global__ __launch_bounds__(kSmallNT) void k_small_rows(const int64_t* __restrict__ values, int n, TableDev t, Work w,
                                                         int64_t* h_live, int64_t tag, int64_t* __restrict__ rows_out,
                                                         int64_t* n_inserted) {
  constexpr int NT = kSmallNT, PT = kSmallPT, NW = NT / kWave;
  static_assert(PT == 8 && kSmallIds < 1 << 15, "sums of a call fit 16 bits; 8 positions in two 16-byte loads");
  __shared__ unsigned int info[kSmallIds];        // by first position: unique id << 16 | start of its segment
  __shared__ unsigned short lnew[kSmallIds];      // by first position: 1 + rank among the keys not found, or 0
  // hot keys: unique id, segment start, occurrences, first unit
  __shared__ unsigned short hotu[kSmallIds / kLong], hotst[kSmallIds / kLong], hotc[kSmallIds / kLong],
      hotunit[kSmallIds / kLong];
  __shared__ int sh[NW][3];
  __shared__ int64_t newrow[kSmallPart], newkey[kSmallPart];
  __shared__ int nnew;
  int* const err = reinterpret_cast<int*>(&t.scal[kTErr]);
  const int64_t* const tsc = small_scalars(w);
  const uint32_t* const counts = small_counts(w);
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wid = tid / kWave;
  // positions 8 tid ... 8 tid + 7: the first occurrences among them
  uint32_t cw[PT];
  {
    const int p0 = tid * PT;
    if (p0 + PT <= n) {
      const uint4 a = *reinterpret_cast<const uint4*>(counts + p0);
      const uint4 b = *reinterpret_cast<const uint4*>(counts + p0 + 4);
      cw[0] = a.x; cw[1] = a.y; cw[2] = a.z; cw[3] = a.w;
      cw[4] = b.x; cw[5] = b.y; cw[6] = b.z; cw[7] = b.w;
    } else {
#pragma unroll
      for (int k = 0; k < PT; ++k) cw[k] = p0 + k < n ? counts[p0 + k] : 0u;
    }
  }
  // this block's ids, one per thread (kSmallPart of them)
  const int i = blockIdx.x * kSmallPart + tid;
  const bool act = tid < kSmallPart && i < n;
  const uint32_t ow = act ? w.occ_word[i] : kOccRejected;
  const int f = ow == kOccRejected ? -1 : static_cast<int>(ow >> 16);
  const int64_t found = f >= 0 ? w.occ_row[f] : -1;  // another block may store the same row there (not for a new key)
  const int own = act ? static_cast<int>(counts[i] & 0xFFFFu) : 0;
  const unsigned long long e = act ? static_cast<unsigned long long>(values[i]) ^ kSign : kEncEmpty;
  const int64_t hw = tsc[kTLive], keys = tsc[kTKeys], F = tsc[kTFree];
  const int64_t tcap[3] = {tsc[kTLimit], tsc[kTRowCap], tsc[kTTomb]};
  if (tid == 0) nnew = 0;
  // occurrences | keys << 16; units | hot keys << 16; keys not found
  int v[3] = {0, 0, 0};
#pragma unroll
  for (int k = 0; k < PT; ++k) {
    const int c = static_cast<int>(cw[k] & 0xFFFFu);
    v[0] += c + (c > 0 ? 1 << 16 : 0);
    if (c > kLong) v[1] += unit_count(c, w.maxu) + (1 << 16);
    v[2] += cw[k] >> 31;
  }
  int inc[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) inc[a] = wave_incl_scan(v[a]);
  if (lane == kWave - 1) {
#pragma unroll
    for (int a = 0; a < 3; ++a) sh[wid][a] = inc[a];
  }
  __syncthreads();
  int ex[3], tot[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {  // every wave sums the waves before it
    int before = 0, all = 0;
    for (int q = 0; q < NW; ++q) {
      before += q < wid ? sh[q][a] : 0;
      all += sh[q][a];
    }
    ex[a] = before + inc[a] - v[a];
    tot[a] = all;
  }
#pragma unroll
  for (int k = 0; k < PT; ++k) {
    const int c = static_cast<int>(cw[k] & 0xFFFFu);
    if (c == 0) continue;
    const int p = tid * PT + k;
    info[p] = static_cast<unsigned int>(ex[0]);
    ex[0] += c + (1 << 16);
    lnew[p] = cw[k] >> 31 ? static_cast<unsigned short>(ex[2] + 1) : 0;
    ex[2] += cw[k] >> 31;
    if (c > kLong) {
      const int q = ex[1] >> 16;
      hotu[q] = static_cast<unsigned short>(info[p] >> 16);
      hotst[q] = static_cast<unsigned short>(info[p] & 0xFFFFu);
      hotc[q] = static_cast<unsigned short>(c);
      hotunit[q] = static_cast<unsigned short>(ex[1] & 0xFFFF);
      ex[1] += unit_count(c, w.maxu) + (1 << 16);
    }
  }
  const int nhot = tot[1] >> 16, nunits = tot[1] & 0xFFFF;
  const Reservation res = reservation(tot[2], hw, keys, F, tcap);
  if (blockIdx.x == 0 && tid == 0) {
    store_reservation(w.scal, t.scal, tot[2], keys, res);
    w.scal[kCU] = tot[0] >> 16;
    w.scal[kCValid] = tot[0] & 0xFFFF;
    w.scal[kCNewReq] = tot[2];
    w.scal[kCNLong] = nhot;
    w.scal[kCNUnits] = nunits;
    if (tot[2] > res.ins) atomicOr(err, kErrFull);
    if (n_inserted) *n_inserted = res.ins;
  }
  __syncthreads();
  int64_t r = found;
  unsigned int x = 0u;
  if (f >= 0) {
    x = info[f];
    const int64_t q = static_cast<int64_t>(lnew[f]) - 1;
    // the first `take` new keys take free rows from the top of the stack
    if (q >= 0) r = q >= res.ins ? -1 : q < res.take ? t.free_rows[res.ftop - 1 - q] : res.hw + (q - res.take);
    if (f == i) {  // the key's first occurrence
      const int u = static_cast<int>(x >> 16);
      if (q >= 0 && r >= 0) {
        const int64_t sl = idmap_claim(t, e);
        if (sl >= 0) {
          t.slots[sl].row = r;
          const int z = atomicAdd(&nnew, 1);
          newrow[z] = r;
          newkey[z] = static_cast<int64_t>(e ^ kSign);
        } else {
          atomicOr(err, kErrProbe);  // no slot: cannot happen below the key limit
        }
      } else if (r >= 0 && t.meta_off >= 0) {
        // eviction: this call is the key's last lookup
        *reinterpret_cast<uint32_t*>(t.store.row(r) + t.meta_off + 8) = t.clock;
      }
      w.unique[u] = static_cast<int64_t>(e ^ kSign);
      w.rows[u] = r;
      w.useg[u] = Seg{r, static_cast<int>(x & 0xFFFFu), own};
    }
  }
  __syncthreads();
  // the rows of the block's new keys
  for (int z = tid / kInitLanes; z < nnew; z += NT / kInitLanes) init_row(t, newrow[z], newkey[z], tid % kInitLanes);
  if (act) {
    if (OCC) {
      w.inverse[i] = f >= 0 ? static_cast<int>(x >> 16) : -1;
      w.occ_row[i] = r;
      w.occ_ref[i] = -1;  // no gradient row yet: the pool writes them
      w.occ_pos[i] = f >= 0 ? static_cast<int>(x & 0xFFFFu) + static_cast<int>(ow & 0xFFFFu) : -1;
    } else {
      rows_out[i] = r;
    }
  }
  if (OCC && blockIdx.x == 0) {
    for (int q = tid; q < nhot; q += NT) {
      w.long_u[q] = hotu[q];
      w.long_start[q] = hotunit[q];
      w.id_ref[q] = 0;  // (no small batch's gradient rows) the backward's count of the key's finished units
    }
    for (int y = tid; y < nunits; y += NT) {
      int lo = 0, hi = nhot;  // the hot key of unit y: hotunit[lo] <= y < hotunit[lo + 1]
      while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (hotunit[mid] <= y) lo = mid;
        else hi = mid;
      }
      const int c = hotc[lo], usz = kUnit << unit_shift(c, w.maxu), j = y - hotunit[lo];
      w.units[y] = Unit{lo, hotst[lo] + j * usz, hotst[lo] + min((j + 1) * usz, c), 0};
    }
  }
  if (blockIdx.x == 0 && tid == 0) publish_live(h_live, tag, res.published);  // last: a store to host memory
}

__global__ __launch_bounds__(kBlock) void k_clear_counts(Work w, int n) {
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i < n) w.id_ref[i] = 0;
}

hipError_t launch_clear_counts(const Work& w, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  k_clear_counts<<<grid_for(n, kBlock), kBlock, 0, s>>>(w, static_cast<int>(n));
  return hipGetLastError();
}

hipError_t launch_small_front(const int64_t* values, int64_t n, const TableDev& t, const Work& w, bool occ_lists,
                              int64_t* h_live, int64_t tag, int64_t* rows_out, int64_t* n_inserted,
                              hipEvent_t* ev_front, hipEvent_t* ev_rows, hipStream_t s) {
  if (n <= 0 || n > kSmallIds) return hipErrorInvalidValue;
  const int ni = static_cast<int>(n);
  int logG = 0;
  while (kSmallPart << logG < ni) ++logG;
  if (ev_front && ev_front[0]) (void)hipEventRecord(ev_front[0], s);
  k_small_dedup<<<1u << logG, kSmallNT, 0, s>>>(values, ni, logG, t, w);
  if (ev_front && ev_front[1]) (void)hipEventRecord(ev_front[1], s);
  if (ev_rows && ev_rows[0]) (void)hipEventRecord(ev_rows[0], s);
  const unsigned nb = grid_for(n, kSmallPart);
  if (occ_lists) k_small_rows<true><<<nb, kSmallNT, 0, s>>>(values, ni, t, w, h_live, tag, nullptr, nullptr);
  else k_small_rows<false><<<nb, kSmallNT, 0, s>>>(values, ni, t, w, h_live, tag, rows_out, n_inserted);
  if (ev_rows && ev_rows[1]) (void)hipEventRecord(ev_rows[1], s);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// eviction of stale keys
// ---------------------------------------------------------------------------

// Slot index of an encoded key, or -1.
__device__ inline int64_t idmap_slot_of(const TableDev& t, unsigned long long e) {
  uint64_t h = idmap_hash(e) & t.cap_mask;
  for (uint64_t probed = 0; probed <= t.cap_mask; ++probed) {
    const unsigned long long k = t.slots[h].key;
    if (k == e) return static_cast<int64_t>(h);
    if (k == kEncEmpty) return -1;
    h = (h + 1) & t.cap_mask;
  }
  return -1;
}

// Row r holds a key whose age (clock - clock of its last lookup, mod 2^32)
// exceeds max_age.  Rows at or past the high-water mark hold nothing.
__device__ inline bool stale_row(const TableDev& t, int64_t r, int64_t hw, uint32_t max_age, int64_t& key) {
  key = INT64_MIN;
  if (r >= hw) return false;
  const uint8_t* m = t.store.row(r) + t.meta_off;
  key = *reinterpret_cast<const int64_t*>(m);
  const uint32_t seen = *reinterpret_cast<const uint32_t*>(m + 8);
  return key != INT64_MIN && static_cast<uint32_t>(t.clock - seen) > max_age;
}

// Stale rows per block of kEvictRows rows (4 per thread).
__global__ __launch_bounds__(kBlock) void k_evict_count(TableDev t, uint32_t max_age, int32_t* __restrict__ bcount) {
  __shared__ int sh[kBlock / kWave + 1];
  const int64_t hw = t.scal[kTLive];
  int c = 0;
#pragma unroll
  for (int k = 0; k < kEvictRows / kBlock; ++k) {
    int64_t key;
    c += stale_row(t, static_cast<int64_t>(blockIdx.x) * kEvictRows + k * kBlock + threadIdx.x, hw, max_age, key);
  }
  const int tot = block_sum<kBlock>(c, sh);
  if (threadIdx.x == 0) bcount[blockIdx.x] = tot;
}

// One block: exclusive scan of the nb block counts in place (chunks of 1024
// with a running carry); the total goes to bcount[nb].
__global__ __launch_bounds__(1024) void k_evict_scan(int32_t* __restrict__ bcount, int64_t nb) {
  __shared__ int sh[1024 / kWave + 1];
  int carry = 0;
  for (int64_t base = 0; base < nb; base += 1024) {
    const int64_t i = base + threadIdx.x;
    const int v = i < nb ? bcount[i] : 0;
    int tot;
    const int ex = block_excl_scan<1024>(v, sh, tot);
    if (i < nb) bcount[i] = carry + ex;
    carry += tot;
  }
  if (threadIdx.x == 0) bcount[nb] = carry;
}

// The stale rows of a block, in row order: each is pushed on the free stack
// (after the rows already there), its key is cleared and its IDMap slot
// becomes a tombstone.
__global__ __launch_bounds__(kBlock) void k_evict_apply(TableDev t, uint32_t max_age,
                                                        const int32_t* __restrict__ bcount) {
  __shared__ int sh[kBlock / kWave + 1];
  constexpr int K = kEvictRows / kBlock;
  const int64_t hw = t.scal[kTLive];
  const int64_t F0 = t.scal[kTFree];
  // thread tid owns rows r0 + tid*K ... + K-1: row order = thread order
  const int64_t r0 = static_cast<int64_t>(blockIdx.x) * kEvictRows + static_cast<int64_t>(threadIdx.x) * K;
  int64_t key[K];
  bool st[K];
  int c = 0;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    st[k] = stale_row(t, r0 + k, hw, max_age, key[k]);
    c += st[k];
  }
  int tot;
  int pos = block_excl_scan<kBlock>(c, sh, tot);
  const int64_t base = F0 + bcount[blockIdx.x];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    if (!st[k]) continue;
    t.free_rows[base + pos++] = r0 + k;
    *reinterpret_cast<int64_t*>(t.store.row(r0 + k) + t.meta_off) = INT64_MIN;
    const int64_t slot = idmap_slot_of(t, static_cast<unsigned long long>(key[k]) ^ kSign);
    if (slot >= 0) t.slots[slot].key = kEncTomb;
    else atomicOr(reinterpret_cast<int*>(&t.scal[kTErr]), kErrProbe);
  }
}

__global__ void k_evict_finish(int64_t* tscal, const int32_t* bcount, int64_t nb) {
  const int64_t n = bcount[nb];
  tscal[kTFree] += n;
  tscal[kTKeys] -= n;
  tscal[kTTomb] += n;
}

hipError_t launch_evict(const TableDev& t, int64_t rows_prov, uint32_t max_age, int32_t* bcount, hipStream_t s) {
  if (t.meta_off < 0) return hipErrorInvalidValue;
  const int64_t nb = std::max<int64_t>(1, (rows_prov + kEvictRows - 1) / kEvictRows);
  k_evict_count<<<static_cast<unsigned>(nb), kBlock, 0, s>>>(t, max_age, bcount);
  k_evict_scan<<<1, 1024, 0, s>>>(bcount, nb);
  k_evict_apply<<<static_cast<unsigned>(nb), kBlock, 0, s>>>(t, max_age, bcount);
  k_evict_finish<<<1, 1, 0, s>>>(t.scal, bcount, nb);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// compaction of the Blocks after eviction
// ---------------------------------------------------------------------------

// Row r holds a key (eviction writes INT64_MIN into a freed row's key field).
__device__ inline bool row_holds_key(const TableDev& t, int64_t r) {
  return *reinterpret_cast<const int64_t*>(t.store.row(r) + t.meta_off) != INT64_MIN;
}

// Per block of kEvictRows rows below the high-water mark hw: the free rows
// below the live count L ("holes") and the rows at or above L that hold a key
// ("movers").  Thread tid owns rows r0 + tid*K ... (row order = thread order).
__global__ __launch_bounds__(kBlock) void k_compact_count(TableDev t, int64_t L, int64_t hw, int32_t* __restrict__ hc,
                                                          int32_t* __restrict__ mc) {
  __shared__ int sh[kBlock / kWave + 1];
  constexpr int K = kEvictRows / kBlock;
  const int64_t r0 = static_cast<int64_t>(blockIdx.x) * kEvictRows + static_cast<int64_t>(threadIdx.x) * K;
  int h = 0, m = 0;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int64_t r = r0 + k;
    if (r >= hw) continue;
    const bool held = row_holds_key(t, r);
    h += r < L && !held;
    m += r >= L && held;
  }
  const int th = block_sum<kBlock>(h, sh);
  __syncthreads();
  const int tm = block_sum<kBlock>(m, sh);
  if (threadIdx.x == 0) {
    hc[blockIdx.x] = th;
    mc[blockIdx.x] = tm;
  }
}

// The holes and the movers of each block, in row order, at their ranks
// (hc / mc hold the blocks' exclusive prefixes).
__global__ __launch_bounds__(kBlock) void k_compact_list(TableDev t, int64_t L, int64_t hw,
                                                         const int32_t* __restrict__ hc, const int32_t* __restrict__ mc,
                                                         int64_t* __restrict__ hole_at, int64_t* __restrict__ src_at,
                                                         int64_t cap) {
  __shared__ int sh[kBlock / kWave + 1];
  constexpr int K = kEvictRows / kBlock;
  const int64_t r0 = static_cast<int64_t>(blockIdx.x) * kEvictRows + static_cast<int64_t>(threadIdx.x) * K;
  bool hole[K], mover[K];
  int h = 0, m = 0;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int64_t r = r0 + k;
    const bool held = r < hw && row_holds_key(t, r);
    hole[k] = r < hw && r < L && !held;
    mover[k] = r >= L && held;
    h += hole[k];
    m += mover[k];
  }
  int tot;
  int hp = hc[blockIdx.x] + block_excl_scan<kBlock>(h, sh, tot);
  int mp = mc[blockIdx.x] + block_excl_scan<kBlock>(m, sh, tot);
#pragma unroll
  for (int k = 0; k < K; ++k) {  // both lists hold at most cap = hw - L rows
    if (hole[k] && hp < cap) hole_at[hp] = r0 + k;
    if (mover[k] && mp < cap) src_at[mp] = r0 + k;
    hp += hole[k];
    mp += mover[k];
  }
}

// One wave per move: the k-th mover's row (values, state, key and clock)
// is copied into the k-th hole, 16 bytes per lane, and its IDMap slot takes
// the new row.  npairs: the device-side count (the movers' total).
__global__ __launch_bounds__(kBlock) void k_compact_move(TableDev t, const int64_t* __restrict__ hole_at,
                                                         const int64_t* __restrict__ src_at,
                                                         const int32_t* __restrict__ nholes,
                                                         const int32_t* __restrict__ nmovers, int64_t cap) {
  const int lane = threadIdx.x & (kWave - 1);
  // the two counts agree for a consistent table (both are the keys missing
  // below L); the minimum keeps every index inside the lists regardless
  const int64_t np = min(min(static_cast<int64_t>(*nholes), static_cast<int64_t>(*nmovers)), cap);
  if (blockIdx.x == 0 && threadIdx.x == 0 && *nholes != *nmovers)
    atomicOr(reinterpret_cast<int*>(&t.scal[kTErr]), kErrProbe);
  const int words = static_cast<int>(t.store.stride / 16);
  for (int64_t k = static_cast<int64_t>(blockIdx.x) * (kBlock / kWave) + threadIdx.x / kWave; k < np;
       k += static_cast<int64_t>(gridDim.x) * (kBlock / kWave)) {
    const int64_t src = src_at[k], dst = hole_at[k];
    const uint4* sp = reinterpret_cast<const uint4*>(t.store.row(src));
    uint4* dp = reinterpret_cast<uint4*>(t.store.row(dst));
    for (int q = lane; q < words; q += kWave) dp[q] = sp[q];
    if (lane == 0) {
      const int64_t key = *reinterpret_cast<const int64_t*>(t.store.row(src) + t.meta_off);
      const int64_t slot = idmap_slot_of(t, static_cast<unsigned long long>(key) ^ kSign);
      if (slot >= 0) t.slots[slot].row = dst;
      else atomicOr(reinterpret_cast<int*>(&t.scal[kTErr]), kErrProbe);
    }
  }
}

__global__ void k_compact_finish(int64_t* tscal, int64_t L) {
  tscal[kTLive] = L;
  tscal[kTFree] = 0;
}

hipError_t launch_compact_rows(const TableDev& t, int64_t L, int64_t hw, int32_t* hc, int32_t* mc, int64_t* hole_at,
                               int64_t* src_at, hipStream_t s) {
  if (t.meta_off < 0 || hw <= L) return hipErrorInvalidValue;
  const int64_t nb = (hw + kEvictRows - 1) / kEvictRows;
  k_compact_count<<<static_cast<unsigned>(nb), kBlock, 0, s>>>(t, L, hw, hc, mc);
  k_evict_scan<<<1, 1024, 0, s>>>(hc, nb);  // exclusive prefixes; the totals at [nb]
  k_evict_scan<<<1, 1024, 0, s>>>(mc, nb);
  k_compact_list<<<static_cast<unsigned>(nb), kBlock, 0, s>>>(t, L, hw, hc, mc, hole_at, src_at, hw - L);
  k_compact_move<<<grid_for(hw - L, kBlock / kWave, 8192), kBlock, 0, s>>>(t, hole_at, src_at, hc + nb, mc + nb,
                                                                           hw - L);
  k_compact_finish<<<1, 1, 0, s>>>(t.scal, L);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// find-or-insert results, find-only lookups, rehash, export, read-back
// ---------------------------------------------------------------------------

__global__ __launch_bounds__(kBlock) void k_map_rows(const int32_t* __restrict__ inverse, const int64_t* __restrict__ rows,
                                                     int64_t n, int64_t* __restrict__ out, const int64_t* cscal,
                                                     int64_t* n_inserted) {
  const int64_t i = blockIdx.x * static_cast<int64_t>(kBlock) + threadIdx.x;
  if (i == 0 && n_inserted) *n_inserted = cscal[kCNew];
  if (i < n) {
    const int u = inverse[i];
    out[i] = u >= 0 ? rows[u] : -1;
  }
}

hipError_t launch_map_rows(const Work& w, int64_t n, int64_t* rows_out, int64_t* n_inserted, hipStream_t s) {
  k_map_rows<<<grid_for(n, kBlock, 1ll << 31), kBlock, 0, s>>>(w.inverse, w.rows, n, rows_out, w.scal, n_inserted);
  return hipGetLastError();
}

__global__ __launch_bounds__(kBlock) void k_find(TableDev t, const int64_t* __restrict__ keys, int64_t n,
                                                 int64_t* __restrict__ out) {
  for (int64_t i = blockIdx.x * static_cast<int64_t>(kBlock) + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * kBlock) {
    const unsigned long long e = static_cast<unsigned long long>(keys[i]) ^ kSign;
    out[i] = e <= kEncTomb ? -1 : idmap_lookup(t, e);
  }
}

hipError_t launch_find(const TableDev& t, const int64_t* keys, int64_t n, int64_t* rows_out, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  k_find<<<grid_for(n, kBlock, 16384), kBlock, 0, s>>>(t, keys, n, rows_out);
  return hipGetLastError();
}

__global__ __launch_bounds__(kBlock) void k_rehash(const Slot* __restrict__ old, int64_t old_cap, TableDev t) {
  for (int64_t i = blockIdx.x * static_cast<int64_t>(kBlock) + threadIdx.x; i < old_cap;
       i += static_cast<int64_t>(gridDim.x) * kBlock) {
    const Slot sl = old[i];
    if (sl.key <= kEncTomb) continue;
    const int64_t slot = idmap_claim(t, sl.key);
    if (slot >= 0) t.slots[slot].row = sl.row;
    else atomicOr(reinterpret_cast<int*>(&t.scal[kTErr]), kErrProbe);
  }
}

hipError_t launch_rehash(const Slot* old_slots, int64_t old_cap, const TableDev& t, hipStream_t s) {
  k_rehash<<<grid_for(old_cap, kBlock, 65536), kBlock, 0, s>>>(old_slots, old_cap, t);
  return hipGetLastError();
}

__global__ __launch_bounds__(kBlock) void k_export(TableDev t, int64_t cap_slots, int64_t* __restrict__ keys,
                                                   int64_t* __restrict__ rows, int64_t cap, unsigned long long* counter) {
  for (int64_t i = blockIdx.x * static_cast<int64_t>(kBlock) + threadIdx.x; i < cap_slots;
       i += static_cast<int64_t>(gridDim.x) * kBlock) {
    const Slot sl = t.slots[i];
    if (sl.key <= kEncTomb) continue;
    const unsigned long long k = atomicAdd(counter, 1ull);
    if (static_cast<int64_t>(k) < cap) {
      keys[k] = static_cast<int64_t>(sl.key ^ kSign);
      rows[k] = sl.row;
    }
  }
}

__global__ void k_copy_scalar(const int64_t* src, int64_t* dst) { *dst = *src; }

hipError_t launch_export(const TableDev& t, int64_t cap_slots, int64_t* keys, int64_t* rows, int64_t cap,
                         int64_t* n_dev, hipStream_t s) {
  (void)hipMemsetAsync(&t.scal[kTExport], 0, sizeof(int64_t), s);
  k_export<<<grid_for(cap_slots, kBlock, 65536), kBlock, 0, s>>>(
      t, cap_slots, keys, rows, cap, reinterpret_cast<unsigned long long*>(&t.scal[kTExport]));
  if (n_dev) k_copy_scalar<<<1, 1, 0, s>>>(&t.scal[kTExport], n_dev);
  return hipGetLastError();
}

// Row read-back: a lane group of D / 4 lanes takes kReadRows rows at a time,
// each lane 4 consecutive elements of w and of every state vector.  Random
// row reads and a streamed output bound it, so all of a lane's 16-byte loads
// (8 for bf16 w) are issued before the first store, and the output leaves
// with non-temporal 16-byte stores.  A row-wise state row (its length is not
// a multiple of 4 floats) or an output that is not 16-byte aligned is stored
// float by float.  Measured for 1.45M rows of dim 64 fp32 with Adam state
// (2.2 GB read and written): 388 us, 5.7 TB/s; one thread per element (4-byte
// accesses, a row-id load and a division each) took 582 us.  3.77M bf16 rows
// of dim 32 with Adagrad state: 556 -> 299 us.
constexpr int kReadRows = 2;

__device__ inline void store_out4(float* p, const float4& v, bool vec) {
  if (vec) {
    const nt_f32x4 a = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(a, reinterpret_cast<nt_f32x4*>(p));
  } else {
    p[0] = v.x;
    p[1] = v.y;
    p[2] = v.z;
    p[3] = v.w;
  }
}

template <int LANES, bool BF16>
__global__ __launch_bounds__(kBlock) void k_read_rows(TableDev t, const int64_t* __restrict__ rows, int64_t n,
                                                      float* __restrict__ w_out, float* __restrict__ state_out,
                                                      bool wvec, bool svec) {
  constexpr int D = LANES * 4;
  constexpr int GPB = kBlock / LANES;
  const int lane = threadIdx.x % LANES, grp = threadIdx.x / LANES;
  const int64_t live = t.scal[kTLive];
  const int se = t.nstate * D + t.rowscalar;
  const float nanv = __builtin_nanf("");
  const float4 nan4 = make_float4(nanv, nanv, nanv, nanv);
  for (int64_t i0 = (static_cast<int64_t>(blockIdx.x) * GPB + grp) * kReadRows; i0 < n;
       i0 += static_cast<int64_t>(gridDim.x) * GPB * kReadRows) {
    int64_t r[kReadRows];
#pragma unroll
    for (int k = 0; k < kReadRows; ++k) {
      r[k] = i0 + k < n ? rows[i0 + k] : -1;
      if (r[k] >= live) r[k] = -1;
    }
    float4 w[kReadRows], s1[kReadRows], s2[kReadRows];
    float sr[kReadRows];
#pragma unroll
    for (int k = 0; k < kReadRows; ++k) {
      w[k] = s1[k] = s2[k] = nan4;
      sr[k] = nanv;
      if (r[k] < 0) continue;
      const uint8_t* rp = t.store.row(r[k]);
      if (w_out) {
        if (BF16) {
          const uint2 h = *reinterpret_cast<const uint2*>(rp + lane * 8);
          w[k] = make_float4(__uint_as_float(h.x << 16), __uint_as_float(h.x & 0xFFFF0000u),
                             __uint_as_float(h.y << 16), __uint_as_float(h.y & 0xFFFF0000u));
        } else {
          w[k] = *reinterpret_cast<const float4*>(rp + lane * 16);
        }
      }
      if (state_out) {
        const float* sp = reinterpret_cast<const float*>(rp + D * (BF16 ? 2 : 4));
        if (t.nstate >= 1) s1[k] = *reinterpret_cast<const float4*>(sp + lane * 4);
        if (t.nstate == 2) s2[k] = *reinterpret_cast<const float4*>(sp + D + lane * 4);
        if (t.rowscalar) sr[k] = sp[t.nstate * D];
      }
    }
#pragma unroll
    for (int k = 0; k < kReadRows; ++k) {
      const int64_t i = i0 + k;
      if (i >= n) break;
      if (w_out) store_out4(w_out + i * D + lane * 4, w[k], wvec);
      if (state_out) {
        float* so = state_out + i * se;
        if (t.nstate >= 1) store_out4(so + lane * 4, s1[k], svec);
        if (t.nstate == 2) store_out4(so + D + lane * 4, s2[k], svec);
        if (t.rowscalar && lane == 0) so[t.nstate * D] = sr[k];
      }
    }
  }
}

template <int LANES>
static void read_rows_dim(const TableDev& t, const int64_t* rows, int64_t n, float* w_out, float* state_out,
                          hipStream_t s) {
  const bool wvec = reinterpret_cast<uintptr_t>(w_out) % 16 == 0;
  const bool svec = reinterpret_cast<uintptr_t>(state_out) % 16 == 0 && !t.rowscalar;
  // one pass over the rows (a grid-stride loop only past 2^31 threads)
  const unsigned g = grid_for(n, static_cast<int64_t>(kBlock / LANES) * kReadRows, int64_t(1) << 23);
  if (t.row_dtype) k_read_rows<LANES, true><<<g, kBlock, 0, s>>>(t, rows, n, w_out, state_out, wvec, svec);
  else k_read_rows<LANES, false><<<g, kBlock, 0, s>>>(t, rows, n, w_out, state_out, wvec, svec);
}

hipError_t launch_read_rows(const TableDev& t, const int64_t* rows, int64_t n, float* w_out, float* state_out,
                            hipStream_t s) {
  if (n <= 0) return hipSuccess;
  switch (t.dim / 4) {
    case 2: read_rows_dim<2>(t, rows, n, w_out, state_out, s); break;
    case 4: read_rows_dim<4>(t, rows, n, w_out, state_out, s); break;
    case 8: read_rows_dim<8>(t, rows, n, w_out, state_out, s); break;
    case 16: read_rows_dim<16>(t, rows, n, w_out, state_out, s); break;
    case 32: read_rows_dim<32>(t, rows, n, w_out, state_out, s); break;
    case 64: read_rows_dim<64>(t, rows, n, w_out, state_out, s); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace rs
