// What lies behind which matrix instruction (TICK) of a unit, for kernels that are ordered instruction by instruction: tables filled at
// compile time.
//
// A 16x16x32 instruction takes the matrix pipe 16 cycles and about 6 to issue, a 32x32x16 one 32 and 4; what lies behind it takes the
// costs below, measured with one wavefront on the SIMD.  Where that is longer than the pipe's share, the pipe waits, and fewer instructions
// behind the next one do not make up for it: so every tick is to take about the same time.  (The forward at d = 64, with two wavefronts per SIMD
// that fill one another's gaps, is dealt by the same costs; others have not been measured there.)
#pragma once

namespace vsa {

template <int TICKS>
struct TickCycles {
  static constexpr int T = TICKS;
  enum Op { MUL, EXP, ADD, CVT };  // of an item, a pair of values: arithmetic on value i, its exponential, a sum, the conversion of the pair
  struct Work {
    Op op;
    int item, i;
  };
  static constexpr int kRead = 8, kWait = 4, kCopy = 8, kScalar = 4;
  static constexpr int cost(Op op) { return op == EXP ? 9 : 5; }

  int cycles[T] = {};  // of what lies behind tick t so far

  // `ops` operations dealt to the ticks from .. to - 1 so that all of them take about the same time; ahead[t]: those ahead of tick t
  constexpr void deal(int (&ahead)[T + 1], const Work* w, int ops, int from, int to) {
    int total = 0, sum = 0, n = 0;
    for (int t = from; t < to; ++t) total += cycles[t];
    for (int i = 0; i < ops; ++i) total += cost(w[i].op);
    for (int t = 0; t < T; ++t) {
      ahead[t] = n;
      if (t < from || t >= to) continue;
      sum += cycles[t];
      while (n < ops && (t == to - 1 || (sum + cost(w[n].op) / 2) * (to - from) <= total * (t - from + 1))) {
        cycles[t] += cost(w[n].op);
        sum += cost(w[n++].op);
      }
    }
    ahead[T] = n;
  }
  // An operation lies behind those of its item that it needs.
  static constexpr bool ordered(const Work* w, int ops) {
    for (int a = 0; a < ops; ++a)
      for (int b = a + 1; b < ops; ++b) {
        if (w[a].item != w[b].item) continue;
        const bool same = w[a].i == w[b].i;
        if (w[a].op == EXP && w[b].op == MUL && same) return false;
        if (w[a].op == ADD && (w[b].op == EXP || w[b].op == MUL) && same) return false;
        if (w[a].op == CVT && (w[b].op == EXP || w[b].op == MUL)) return false;
      }
    return true;
  }
};

// With the reads of LDS and the waits for them.
template <int TICKS, int READS>
struct TickTable : TickCycles<TICKS> {
  static constexpr int T = TICKS, N = READS;
  using TickCycles<TICKS>::cycles;
  struct Read {
    int tick, use;  // behind which instruction it is requested, ahead of which one it is waited for (T and more: of the next unit)
    int kind, i, part;
  };

  Read r[N] = {};
  int issued[T + 1] = {};  // reads ahead of tick t
  int newer[T] = {};       // of those, how many are behind the last one that it needs; -1: it needs none that an earlier tick has not

  // (r is filled)
  constexpr void order_reads() {
    for (int i = 1; i < N; ++i)
      for (int j = i; j > 0 && r[j].tick < r[j - 1].tick; --j) {
        const Read x = r[j];
        r[j] = r[j - 1];
        r[j - 1] = x;
      }
    for (int t = 0; t < T; ++t) {
      for (int i = 0; i < N; ++i) issued[t + 1] += r[i].tick <= t;
      int last = -1;
      for (int i = 0; i < N; ++i)
        if (r[i].use % T == t) last = i;
      newer[t] = last < 0 ? -1 : issued[t] - last - 1 + (r[last].use == t ? 0 : N);
      cycles[t] += this->kRead * (issued[t + 1] - issued[t]) + (newer[t] >= 0 ? this->kWait : 0);
    }
  }
};

}  // namespace vsa
