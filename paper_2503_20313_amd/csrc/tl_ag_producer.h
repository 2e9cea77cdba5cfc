// AllGather side shared by the operators that gather row shards (AG+GEMM, AG+gather+grouped GEMM):
// producer-tile queue, producers, and the consumer wait that helps producing.  gfx950 only.
#pragma once
#include "tl_device.h"

namespace tl {

struct AgProducer {
  const bf16_t* shards[kMaxWorld];  // shard q = rows [q*rows_per_rank, (q+1)*rows_per_rank), each [rows_per_rank, ld]
  bf16_t* gathered;                 // [R*rows_per_rank, ld]
  int ld;                           // row length in elements (K of AG+GEMM, H of the MoE token buffer)
  int R, rank;
  int first_src;                    // source rank whose tiles head the queue; the queue then follows the ring
  int n_ptm_all;                    // row tiles of the whole gathered matrix (ring wrap-around)
  int Tm_p, Tn_p, n_ptm, n_ptn;     // producer tile and the number of tiles in the queue along rows / columns
  int rows_per_rank, rows_per_channel;
  int local_in_place;
  int k_chunks;                     // 1: one flag per channel.  > 1: n_ptn == k_chunks column tiles, one flag per (channel,
                                    // column tile) at flags[channel*k_chunks + tn], and the queue hands out column tile 0
                                    // of every row tile before column tile 1 (a consumer can start on the first K chunk)
  int interleave;                   // 0: the queue takes one source rank after the other.  1: the shard of first_src goes first
                                    // as a whole (the local one under the rotated orders); then row tile j of every other
                                    // rank comes before row tile j+1 of any, the order in which concurrent links deliver.
                                    // Needs at least two source ranks in the queue.
  unsigned pace_q8;                 // 0, or 256 x the ticks of the 100 MHz clock a link needs for one producer tile: a tile of
                                    // a remote shard is then not copied before its last byte would have arrived
  unsigned long long* pace_word;    // (epoch tag << 40 | start time) of the call in flight, set by its first producer
  unsigned epoch;
  unsigned wait_target;             // epoch * expected
  unsigned* flags;                  // [R*C*k_chunks]
  unsigned* ticket;                 // producer-tile queue head (grows by n_ptm*n_ptn per call)
  unsigned share_patience;          // gather by shares: ticks of the 100 MHz clock before a consumer fetches its rows itself
  unsigned ticket_end;              // epoch * number of tickets per call (producer tiles + pushes)
  int n_out;                        // push mode: tickets n_ptm*n_ptn .. +n_out-1 each push one producer tile of the LOCAL shard
                                    // into one peer's copy of the gathered matrix (tile_push_data) and notify that peer
  bf16_t* peer_slots[kMaxWorld];    // where this rank's shard lands at peer q, [rows_per_rank, ld]; entry `rank` unused
  unsigned* pushed;                 // [R * channels per rank]: this rank's rows of channel c pushed into peer q at q*cpr + c
  WaitCtl ctl;
};

// ======================================================================================
// AllGather producer (pull mode).  Producer tiles form a queue that is consumed through an atomic
// ticket counter: ticket i is producer tile (tm, tn) in ring order over source ranks (by default
// rank+1, rank+2, ..., the local shard last).  Whoever holds a ticket copies that tile of the gathered
// matrix from its owner's shard and then notifies the tile's channel.  Dedicated producer
// workgroups drain the queue, and a GEMM workgroup whose channel is not ready yet takes tickets
// too instead of idling, so a consumer can never wait for a producer that is not resident.
// ======================================================================================
// Start time of the call in flight on the 100 MHz clock (low 40 bits), agreed on by all producers: the first one to
// find another call's tag in the word replaces it with this call's tag and its own clock reading.  One lane of wave 0
// of a workgroup tries the compare-and-swap (whichever workgroup's lands first wins); everybody then reads the word
// until it carries this call's tag.  Every branch is wave-uniform for the compiler too.
__device__ __forceinline__ unsigned long long pace_start(const AgProducer& p) {
  const unsigned long long mask40 = (1ull << 40) - 1, tag = (unsigned long long)(p.epoch & 0xffffffu) << 40;
  unsigned long long cur = uniform64(__hip_atomic_load(p.pace_word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
  if ((cur & ~mask40) != tag) {
    if (__builtin_amdgcn_readfirstlane(threadIdx.x >> 6) == 0) lane0_cas64(p.pace_word, cur, tag | ((unsigned long long)wall_clock64() & mask40));
    // bounded: a caller that lets two calls share the workspace at the same time gets no pacing rather than a hang
    int tries = 0;
    do {
      cur = uniform64(__hip_atomic_load(p.pace_word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    } while ((cur & ~mask40) != tag && ++tries < 4096);
    if ((cur & ~mask40) != tag) cur = 0;  // "started long ago": every tile is due
  }
  return cur & mask40;
}

// Called by every lane of one wave; the result is wave-uniform.
__device__ __forceinline__ bool claim_ticket(const AgProducer& p, unsigned* out) {
  const unsigned count = (unsigned)(p.n_ptm * p.n_ptn + p.n_out);
  unsigned t = lane0_fetch_add(p.ticket, 1u);
  unsigned idx = t - (p.ticket_end - count);
  // outside this call's range: the queue is empty (or the counter does not belong to this epoch, e.g. a workspace that
  // was not zeroed): give the ticket back; an index outside [0, count) is never handed out
  if (idx >= count) {
    lane0_add(p.ticket, 0xffffffffu);
    return false;
  }
  *out = idx;
  return true;
}

// Where ticket i lies: row tile tm (of the whole gathered matrix), column tile tn, source rank, channel.
struct ProducerPlace { int tm, tn, src, channel; };
__device__ __forceinline__ ProducerPlace producer_place(const AgProducer& p, int i) {
  const int ptm_per_rank = p.rows_per_rank / p.Tm_p;
  int tmi, tn;
  if (p.k_chunks > 1) { tn = i / p.n_ptm; tmi = i - tn * p.n_ptm; }
  else { tmi = i / p.n_ptn; tn = i - tmi * p.n_ptn; }
  int tm;
  if (p.interleave && tmi >= ptm_per_rank) {
    const int others = p.n_ptm / ptm_per_rank - 1;
    int r = tmi - ptm_per_rank, jm = r / others, s = r - jm * others;
    int q = p.first_src + 1 + s;
    if (q >= p.R) q -= p.R;
    tm = q * ptm_per_rank + jm;
  } else {
    tm = tmi + p.first_src * ptm_per_rank;  // ring order over source ranks: first_src, first_src+1, ...
    if (tm >= p.n_ptm_all) tm -= p.n_ptm_all;
  }
  return {tm, tn, tm / ptm_per_rank /* f_R */, tm / (p.rows_per_channel / p.Tm_p) /* f_C */};
}

__device__ __forceinline__ unsigned* producer_flag(const AgProducer& p, const ProducerPlace& t) {
  return p.flags + (p.k_chunks > 1 ? t.channel * p.k_chunks + t.tn : t.channel);
}

// Starts the copy of a producer tile (nothing to do for the local shard in place); the stores may still be on their way.
template <int DEPTH>
__device__ __forceinline__ void copy_producer_tile(const AgProducer& p, const ProducerPlace& t, int tid, int nthreads) {
  if (t.src == p.rank && p.local_in_place) return;
  const int row_lo = t.tm * p.Tm_p;
  const bf16_t* s = p.shards[t.src] + (long)(row_lo - t.src * p.rows_per_rank) * p.ld + (long)t.tn * p.Tn_p;
  bf16_t* d = p.gathered + (long)row_lo * p.ld + (long)t.tn * p.Tn_p;
  copy_tile<DEPTH>(s, p.ld, d, p.ld, p.Tm_p, p.Tn_p, tid, nthreads);
}

// All threads of the workgroup call this with the same ticket index; `wave` is the wave-uniform wave index.
// DEPTH = loads in flight per lane of the copy.
template <int DEPTH>
__device__ __forceinline__ void produce_tile(const AgProducer& p, int i, int tid, int wave, int nthreads) {
  const ProducerPlace t = producer_place(p, i);
  if (p.pace_q8 && t.src != p.rank) {
    // the links of all source ranks run side by side; this tile is number `nth` of what its rank sends
    const int ptm_per_rank = p.rows_per_rank / p.Tm_p, jm = t.tm - t.src * ptm_per_rank;
    const int nth = p.k_chunks > 1 ? t.tn * ptm_per_rank + jm : jm * p.n_ptn + t.tn;
    const unsigned long long due = ((unsigned long long)(nth + 1) * p.pace_q8) >> 8;
    const unsigned long long t0 = pace_start(p);
    while ((((unsigned long long)wall_clock64() - t0) & ((1ull << 40) - 1)) < due) __builtin_amdgcn_s_sleep(8);
  }
  copy_producer_tile<DEPTH>(p, t, tid, nthreads);
  wait_all_vmem();  // this wave's written-through stores are complete ...
  __syncthreads();  // ... and so are every other wave's: the tile is where every die sees it
  if (wave == 0) lane0_add(producer_flag(p, t), 1u);
}

// ======================================================================================
// The gather as shares, for launches that are one round of workgroups (a queue hands out tiles at 11 ns each -- adds to one
// address follow one another -- and costs every workgroup several trips to memory per tile: 20 us before the first tile of
// [512,8192] x [8192,3584] could start, 8 us as shares): workgroup `part` of `parts` copies tickets [lo, hi) x part / parts,
// all copies in flight together, and notifies once per channel.  A workgroup that is not on the chip keeps its share back;
// consumer_wait_shared helps itself after a while, so nobody depends on it for good.
// ======================================================================================
template <int DEPTH>
__device__ __forceinline__ void gather_share(const AgProducer& p, int lo, int hi, int part, int parts, int tid, int nthreads) {
  const int first = lo + (int)((long)(hi - lo) * part / parts), end = lo + (int)((long)(hi - lo) * (part + 1) / parts);
  if (first >= end) return;
  for (int i = first; i < end; i++) copy_producer_tile<DEPTH>(p, producer_place(p, i), tid, nthreads);
  wait_all_vmem();
  __syncthreads();   // every wave's written-through stores are complete
  if (__builtin_amdgcn_readfirstlane(tid >> 6) == 0) {
    unsigned* flag = producer_flag(p, producer_place(p, first));
    unsigned n = 1;
    for (int i = first + 1; i < end; i++) {
      unsigned* f = producer_flag(p, producer_place(p, i));
      if (f != flag) { lane0_add(flag, n); flag = f; n = 0; }
      n++;
    }
    lane0_add(flag, n);
  }
}

// consumer_tile_wait on a gather by shares: all channels' flags in one look (lane c polls channel c).  After
// p.share_patience ticks without them the workgroup copies the missing rows itself -- the same bytes, so it does not matter
// that their owner copies and notifies them as well once it runs -- and goes on.  The patience covers the gather itself, or
// all workgroups of a long one would start over with it together ([65536,8192] at 8 ranks: 1 GiB, 4.7 ms instead of 0.8);
// and before each piece the channel is looked at again, for owners that were merely late.  With K chunks this is about the
// first chunk only: the others are copied by the workgroups at the front of the grid, which start before any workgroup that
// waits and wait for nobody themselves.
template <int DEPTH>
__device__ __forceinline__ void consumer_wait_shared(const AgProducer& p, unsigned long long chan_mask, int tid, int nthreads, int* s_state) {
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int first = __builtin_ctzll(chan_mask);
  unsigned long long missing = 0;
  if (wave == 0) {
    const unsigned long long t0 = wall_clock64();
    const bool mine = (chan_mask >> lane) & 1ull;
    int give_up = 0;
    for (;;) {
      const unsigned f = __hip_atomic_load(p.flags + (mine ? lane : first) * p.k_chunks, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      missing = __builtin_amdgcn_ballot_w64(mine && (int)(f - p.wait_target) < 0);
      if (!missing) break;
      const unsigned long long waited = wall_clock64() - t0;
      if (waited > p.share_patience) { give_up = 1; break; }
      __builtin_amdgcn_s_sleep(2);
    }
    *s_state = give_up;
    s_state[1] = (int)(unsigned)missing;
    s_state[2] = (int)(unsigned)(missing >> 32);
  }
  __syncthreads();
  if (__builtin_amdgcn_readfirstlane(*s_state)) {
    missing = (unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane(s_state[1]) | ((unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane(s_state[2]) << 32);
    const int rows = p.rows_per_channel, cols = p.k_chunks > 1 ? p.Tn_p : p.ld;
    for (; missing; missing &= missing - 1) {
      const int ch = __builtin_ctzll(missing), row_lo = ch * rows, src = row_lo / p.rows_per_rank;
      if (src == p.rank && p.local_in_place) continue;
      for (int r = 0; r < rows; r += p.Tm_p) {   // (a piece of a tile mover spans less than 2 GiB)
        if (wave == 0) *s_state = (int)(__hip_atomic_load(p.flags + ch * p.k_chunks, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - p.wait_target) >= 0;
        __syncthreads();
        const int arrived = __builtin_amdgcn_readfirstlane(*s_state);
        __syncthreads();
        if (arrived) break;
        copy_tile<DEPTH>(p.shards[src] + (long)(row_lo + r - src * p.rows_per_rank) * p.ld, p.ld, p.gathered + (long)(row_lo + r) * p.ld, p.ld, p.Tm_p, cols, tid,
                         nthreads);
      }
    }
    wait_all_vmem();
  }
  acquire_after_wait(p.ctl);
  __syncthreads();
}

// Push mode (paper: "Data Primitives", push mode): ticket j of the push range is producer tile j % (tiles per shard) of the local shard,
// bound for peer rank+1+j/(tiles per shard).  The tile is written into that peer's copy of the gathered matrix and the
// peer's channel counter is raised (peer_tile_notify; here: the pushed counters).
template <int DEPTH>
__device__ __forceinline__ void push_tile(const AgProducer& p, int j, int tid, int wave, int nthreads) {
  const int tiles_per_shard = (p.rows_per_rank / p.Tm_p) * p.n_ptn;
  const int d = j / tiles_per_shard, t = j - d * tiles_per_shard;
  int q = p.rank + 1 + d;
  if (q >= p.R) q -= p.R;
  const int tm = t / p.n_ptn, tn = t - tm * p.n_ptn;
  const long off = (long)tm * p.Tm_p * p.ld + (long)tn * p.Tn_p;
  copy_tile<DEPTH>(p.shards[p.rank] + off, p.ld, p.peer_slots[q] + off, p.ld, p.Tm_p, p.Tn_p, tid, nthreads);
  wait_all_vmem();
  __syncthreads();  // every wave's written-through stores are complete
  const int cpr = p.rows_per_rank / p.rows_per_channel;
  if (wave == 0) lane0_add(p.pushed + q * cpr + (tm * p.Tm_p) / p.rows_per_channel, 1u);
}

// A claimed ticket of either kind.
template <int DEPTH>
__device__ __forceinline__ void work_ticket(const AgProducer& p, int i, int tid, int wave, int nthreads) {
  const int n_in = p.n_ptm * p.n_ptn;
  if (i < n_in) produce_tile<DEPTH>(p, i, tid, wave, nthreads);
  else push_tile<DEPTH>(p, i - n_in, tid, wave, nthreads);
}

// Every branch in the two loops below is wave-uniform for the compiler too (see lane0_fetch_add).
__device__ __forceinline__ void ag_producer(const AgProducer& p, int tid, int nthreads, int* s_ticket) {
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  for (;;) {
    if (wave == 0) {
      unsigned t;
      int v = claim_ticket(p, &t) ? (int)t : -1;
      *s_ticket = v;  // all lanes of wave 0 store the same value
    }
    __syncthreads();
    int i = __builtin_amdgcn_readfirstlane(*s_ticket);
    __syncthreads();
    if (i < 0) break;
    work_ticket<8>(p, i, tid, wave, nthreads);
  }
}

// consumer_tile_wait for the channels set in chan_mask (bit = global channel index; with K chunks: their first chunk) by a whole workgroup: while a channel is short of its target
// the workgroup works off producer tickets; with the queue empty it sleeps and polls (bounded by ctl.timeout).
// DEPTH = loads in flight per lane when this workgroup copies a producer tile itself: deep where the caller's registers allow
// (a ticket then takes a quarter of the time), shallow where they are full.
// ONE: the mask has a single channel (a kernel whose registers are full saves the lane arithmetic).
template <int DEPTH = 2, bool ONE = false>
__device__ __forceinline__ void consumer_wait_or_produce(const AgProducer& p, unsigned long long chan_mask, int tid, int nthreads, int* s_ticket) {
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int first = ONE || chan_mask ? __builtin_ctzll(chan_mask) : 0;   // (no channel: nothing to wait for, but a flag to look at)
  unsigned long long t0 = 0;
  if (wave == 0 && (p.ctl.timeout || p.pace_q8)) t0 = wall_clock64();
  // Tickets are taken only while the queue head has not passed the last tile of the awaited channels: beyond that point every
  // tile this workgroup needs is already in the hands of a resident workgroup, and taking more tickets would only delay it.
  int limit = 0;
  {
    const int tpc = p.rows_per_channel / p.Tm_p, ptm_per_rank = p.rows_per_rank / p.Tm_p;
    for (unsigned long long m = chan_mask; m; m &= m - 1) {
      int qi, qn;  // queue position (in row tiles) of the channel's first row tile, and of the one after its last
      const int ch0 = __builtin_ctzll(m), cpr = ptm_per_rank / tpc;
      if (p.interleave && ch0 / cpr != p.first_src) {
        const int others = p.n_ptm / ptm_per_rank - 1, c = ch0 % cpr;
        int s = ch0 / cpr - p.first_src - 1;
        if (s < 0) s += p.R;
        qi = ptm_per_rank + c * tpc * others + s;
        qn = ptm_per_rank + ((c + 1) * tpc - 1) * others + s + 1;
      } else {
        qi = __builtin_ctzll(m) * tpc - p.first_src * ptm_per_rank;
        if (qi < 0) qi += p.n_ptm_all;
        qn = qi + tpc;
      }
      int end = p.k_chunks > 1 ? qn : qn * p.n_ptn;  // with K chunks: the channel's tiles of chunk 0
      limit = end > limit ? end : limit;
    }
  }
  // With simulated links a ticket is a tile that may not be due for a long time: a consumer that took one would sleep on
  // it while its own rows arrive, and more workers do not make a link faster.  It only waits -- unless nothing has come
  // for far longer than a link takes (a millisecond): then no producer is running beside this kernel (a tool that runs
  // kernels one at a time, say), and the consumers work the queue off themselves as they do without links.
  const unsigned long long patience = p.pace_q8 ? 100000ull : 0ull;
  const unsigned queue_begin = p.ticket_end - (unsigned)(p.n_ptm * p.n_ptn + p.n_out);
  for (;;) {
    if (wave == 0) {
      // one round trip for all channels: lane c looks at channel c (lanes of other channels at the first awaited one).  The
      // queue head, which the producers keep adding to, is read only by who still misses something: read along with the
      // flags it cost attention, whose waits mostly find their rows there, 3 % (S=3328, 16 heads: 139.6 us, 143.2 so)
      const bool mine = ONE || ((chan_mask >> lane) & 1ull);
      const unsigned f = __hip_atomic_load(p.flags + (mine && !ONE ? lane : first) * p.k_chunks, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const unsigned long long missing = __builtin_amdgcn_ballot_w64(mine && (int)(f - p.wait_target) < 0);
      int state = missing ? -1 : -2;  // -2: ready, -1: not ready and nothing to produce, >= 0: ticket to work off
      const int first_short = ONE ? first : (missing ? __builtin_ctzll(missing) : 0);
      if (state == -1) {
        unsigned t;
        const unsigned head = __builtin_amdgcn_readfirstlane(__hip_atomic_load(p.ticket, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        if ((int)(head - queue_begin) < limit && (!patience || wall_clock64() - t0 > patience) && claim_ticket(p, &t)) state = (int)t;
        else if (p.ctl.timeout) {
          int st = __builtin_amdgcn_readfirstlane(__hip_atomic_load(p.ctl.status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
          if (st != 0) state = -2;  // abandoned elsewhere
          else if (wall_clock64() - t0 > p.ctl.timeout) {
            int expected = 0;  // every lane tries, the first one wins, all carry the same value
            __hip_atomic_compare_exchange_strong(p.ctl.status, &expected, 1 + first_short, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            state = -2;
          }
        }
      }
      *s_ticket = state;
    }
    __syncthreads();
    int state = __builtin_amdgcn_readfirstlane(*s_ticket);
    __syncthreads();
    if (state == -2) break;
    if (state >= 0) work_ticket<DEPTH>(p, state, tid, wave, nthreads);
    else __builtin_amdgcn_s_sleep(8);
  }
  acquire_after_wait(p.ctl);
  __syncthreads();
}


}  // namespace tl
