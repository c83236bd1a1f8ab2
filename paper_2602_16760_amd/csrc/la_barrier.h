// The persistent kernels' grid barrier, what of it is plain C++: which epochs a launch counts from, and when a wait gives up.
#pragma once

#ifdef __HIPCC__
#define LA_HD __host__ __device__
#else
#define LA_HD
#endif

namespace la {

// A wait is patient for a number of units of about a microsecond, four polls each.
constexpr unsigned PATIENCE = 1u << 21, PATIENCE_MOST = (1u << 30) - 2;  // (the most that 32 bits of polls can pass)
inline unsigned barrier_patience(unsigned units) { return units == 0 ? PATIENCE : units < PATIENCE_MOST ? units : PATIENCE_MOST; }
LA_HD inline bool patience_over(unsigned polls, unsigned units) { return (polls >> 2) > units; }
// Whether a wait ends without result after one more poll: its patience is over, or its workgroup is marked dead by another wave (dead(),
// which costs a trip to LDS: looked at every 256 polls, 64 us).  Neither is expected: laid out in the way of the polls the two took
// small_bf16's 15 barriers 0.6 us more.
template <typename Dead>
LA_HD inline bool wait_over(unsigned &polls, unsigned units, Dead dead) {
  return __builtin_expect(patience_over(++polls, units), 0) || (__builtin_expect((polls & 255u) == 0, 0) && dead());
}

// A launch of n barriers passes epochs e + 1 .. e + n and leaves them in the barrier words.  A wait ends on any word that has reached its
// epoch, so what a launch finds there must be below its first.  A captured launch is replayed with the epoch that it was captured
// with: the words are cleared in front of it, in the graph, and it counts from 0.  A launch that is not captured counts on from the
// last one, and always from above the `most` barriers that a replay can leave behind, of which the host knows nothing.
// Words that count arrivals (`counters`: the LDS-ring kernel) have to be right to one: once a launch was captured, every launch clears them.
struct BarrierEpochs {
  static constexpr unsigned RESTART = 1u << 26;  // (far below the words' flag bit)
  unsigned most = 0;  // barriers of the longest launch
  bool counters = false;
  bool captured = false;
  unsigned next = 0;

  struct Launch {
    unsigned epoch0;
    bool clear;  // the words are cleared on the launch's stream in front of it
  };
  void init(unsigned most_, bool counters_) {
    most = most_;
    counters = counters_;
    next = first();
  }
  unsigned first() const { return counters ? 0 : most; }
  Launch launch(unsigned n, bool capturing) {
    captured = captured || capturing;
    if (capturing || (counters && captured)) return {0, true};
    const bool restart = next > RESTART;
    if (restart) next = first();
    const Launch l{next, restart};
    next += n;
    return l;
  }
  // The words are cleared on a stream (capturing: when the graph runs, if ever).
  void cleared(bool capturing) {
    captured = captured || capturing;
    if (!capturing) next = first();
  }
};

}  // namespace la
