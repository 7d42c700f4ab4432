// Host model of the event log's pool: how the waves of a launch share its
// blocks, how large it has to be, and how k_replay_events reads it in tiles.
//
// Waves with random numbers of records (many of them none) run interleaved, as
// they do on the chip.  Each opens its log with its own first block or with one
// handed out (log_own_blocks) and goes on in blocks handed out after those, as
// log_trip and log_close in step.hip do; records carry their wave and number.
// The reader takes tiles of 8 or 16 records, finds the first marker among them
// and never looks past the block's end; what lies behind a wave's end marker is
// left over from other launches and looks like records and markers.
//
// Checked: a pool of exactly log_need (blocks handed out) or log_own_need bytes
// (own first blocks) never runs out; the readers get every wave's records back in
// order; waves without records need nothing; and, step after step with the
// host's rules (grow to 5/4 of the need while the memory's limit allows, keep
// the pool otherwise), a launch that fits the pool by log_need runs out at most
// once before it is replayed.  Own first blocks in a pool of only log_need bytes
// must be seen to run out.
//
// Usage: event_log_pool_model [trials]; exit 0: all of the above.
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "../paper_2409_17299_amd/csrc/event_log.h"

namespace {

using namespace sfqed;

struct Header {
  uint64_t base, tag, wave, number;
};

struct Launch {
  std::vector<uint32_t> recs;  // per wave
  uint32_t slot;               // bytes of a lane's slot
  uint64_t tally() const {
    uint64_t t = 0;
    for (uint32_t r : recs) t += log_tally(r, slot);
    return t;
  }
};

Launch random_launch(std::mt19937_64& rng) {
  Launch l;
  l.slot = rng() % 2 ? 8 : 16;
  const uint32_t per = (uint32_t)log_records_per_block(l.slot);
  l.recs.resize(1 + rng() % 40);
  const int mode = (int)(rng() % 4);  // none at all, few waves, all waves, around block ends
  for (uint32_t& r : l.recs) {
    if (mode == 0) r = 0;
    else if (mode == 1) r = rng() % 8 ? 0 : (uint32_t)(1 + rng() % (4 * per));
    else if (mode == 2) r = (uint32_t)(1 + rng() % (3 * per));
    else r = (uint32_t)((rng() % 4) * (per - 1) + rng() % 3);
  }
  return l;
}

// Runs the launch on `cap` bytes, `own` first blocks belonging to the waves.
// Returns false when the pool ran out; otherwise the heads and the headers.
bool write(const Launch& l, uint64_t cap, uint32_t own, std::mt19937_64& rng, std::vector<uint64_t>& head,
           std::vector<Header>& pool) {
  const uint32_t per = (uint32_t)log_records_per_block(l.slot), waves = (uint32_t)l.recs.size();
  pool.assign(cap / kLogBlock * per, Header{});
  for (Header& h : pool) h = {rng() % 7, rng() % 3, rng() % waves, rng() % 1000};  // left over
  head.assign(waves, 0);
  std::vector<uint64_t> blk(waves, 0);
  std::vector<uint32_t> pos(waves, 0), done(waves, 0);
  std::vector<char> open(waves, 0);
  uint64_t used = 0;
  std::vector<uint32_t> live;
  for (uint32_t w = 0; w < waves; ++w)
    if (l.recs[w]) live.push_back(w);
  while (!live.empty()) {
    const size_t i = rng() % live.size();
    const uint32_t w = live[i];
    if (!open[w] || pos[w] + 1 >= per) {
      uint64_t b = w;
      if (open[w] || !own) b = own + used++;
      if ((b + 1) * kLogBlock > cap) return false;
      if (open[w]) pool[blk[w] * per + pos[w]] = {b * kLogBlock, kLogJump, 0, 0};
      else head[w] = b * kLogBlock + 1;
      open[w] = 1;
      blk[w] = b;
      pos[w] = 0;
    }
    pool[blk[w] * per + pos[w]++] = {0, kLogRecord, w, done[w]};
    if (++done[w] == l.recs[w]) {
      pool[blk[w] * per + pos[w]] = {0, kLogEnd, 0, 0};
      live[i] = live.back();
      live.pop_back();
    }
  }
  return true;
}

// Mistakes of the tiled reader over all waves.
int64_t read(const Launch& l, const std::vector<uint64_t>& head, const std::vector<Header>& pool, int tile) {
  const int per = (int)log_records_per_block(l.slot);
  int64_t bad = 0;
  for (uint32_t w = 0; w < l.recs.size(); ++w) {
    if (!head[w]) {
      bad += l.recs[w] != 0;
      continue;
    }
    uint64_t blk = head[w] - 1, got = 0;
    int pos = 0;
    for (int guard = 0;; ++guard) {
      const int room = std::min(per - pos, tile);
      if (room <= 0 || guard > 1 << 16 || (blk / kLogBlock) * per + pos + room > pool.size()) {
        ++bad;
        break;
      }
      const Header* at = &pool[(blk / kLogBlock) * per + pos];
      int nrec = 0;
      while (nrec < room && at[nrec].tag == kLogRecord) ++nrec;
      for (int t = 0; t < nrec; ++t) bad += at[t].wave != w || at[t].number != got++;
      if (nrec == room) {
        pos += nrec;
      } else if (at[nrec].tag == kLogJump) {
        blk = at[nrec].base;
        pos = 0;
      } else {
        break;
      }
    }
    bad += got != l.recs[w];
  }
  return bad;
}

}  // namespace

int main(int argc, char** argv) {
  const int trials = argc > 1 ? std::atoi(argv[1]) : 300;
  std::mt19937_64 rng(7);
  int64_t bad = 0, ran_out = 0, idle = 0, short_own = 0, jumps = 0;
  std::vector<uint64_t> head;
  std::vector<Header> pool;
  for (int t = 0; t < trials; ++t) {
    const Launch l = random_launch(rng);
    const uint32_t waves = (uint32_t)l.recs.size();
    const uint64_t need = log_need(l.tally()), own_need = log_own_need(l.tally(), waves);
    if (*std::max_element(l.recs.begin(), l.recs.end()) == 0) {
      ++idle;
      bad += need != 0;
    }
    for (uint32_t own : {0u, waves}) {
      if (!write(l, own ? own_need : need, own, rng, head, pool)) {
        ++ran_out;
        continue;
      }
      for (int tile : {8, 16}) bad += read(l, head, pool, tile);
    }
    for (uint32_t r : l.recs) jumps += r >= log_records_per_block(l.slot);
    if (need < own_need) short_own += !write(l, need, waves, rng, head, pool);
  }
  // the host's rules over steps of one to three launches, a few times each
  int64_t refused = 0, twice = 0, own_runs = 0;
  for (int t = 0; t < trials; ++t) {
    const uint64_t limit = kLogBlock * (rng() % 120);  // the most the memory gives
    uint64_t cap = 0, seen_own = 0;
    for (int phase = 0; phase < 3; ++phase) {
      std::vector<Launch> step(1 + rng() % 3);
      for (Launch& l : step) l = random_launch(rng);
      std::vector<int> late(step.size(), 0);
      for (int rep = 0; rep < 4; ++rep) {
        uint64_t need = 0, own_need = 0;
        for (size_t i = 0; i < step.size(); ++i) {
          const Launch& l = step[i];
          const uint32_t waves = (uint32_t)l.recs.size(), own = log_own_blocks(cap, seen_own, waves);
          const bool fits = log_need(l.tally()) <= cap;
          if (write(l, cap, own, rng, head, pool)) {
            own_runs += own != 0;
            bad += read(l, head, pool, 16);
          } else if (fits) {
            twice += ++late[i] > 1;
          }
          need = std::max(need, log_need(l.tally()));
          own_need = std::max(own_need, log_own_need(l.tally(), waves));
        }
        seen_own = std::max(seen_own, own_need);
        if (need > cap) {
          if (need + need / 4 <= limit) cap = need + need / 4;
          else ++refused;
        }
      }
    }
  }
  std::printf("%lld mistakes, %lld exact pools ran out, %lld launches without records, %lld waves over several blocks, "
              "%lld own first blocks without room; steps: %lld launches with own first blocks, %lld pools refused, "
              "%lld launches that fit ran out twice\n",
              (long long)bad, (long long)ran_out, (long long)idle, (long long)jumps, (long long)short_own,
              (long long)own_runs, (long long)refused, (long long)twice);
  return !bad && !ran_out && !twice && idle && jumps && short_own && own_runs && refused ? 0 : 1;
}
