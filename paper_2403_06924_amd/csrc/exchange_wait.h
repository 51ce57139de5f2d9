// How long workgroups that exchange words through memory wait for each other.  Plain arithmetic, also compiled for the host
// by its test.
#ifndef SRQ_EXCHANGE_WAIT_H_
#define SRQ_EXCHANGE_WAIT_H_
#include <cstdint>

#ifdef __HIPCC__
#include <hip/hip_runtime.h>
#define SRQ_ANYWHERE __host__ __device__ __forceinline__
#else
#define SRQ_ANYWHERE inline
#endif

namespace srq {

// The wait of a thread for all words of one exchange.  The time runs from the first word that is not there yet and is not
// given again to the words after it: whoever has run out of it reads the rest as they are, since one word that is missing
// makes a workgroup work out all of them.
struct ExchangeWait {
  uint32_t ticks;
  uint64_t until = 0;                                  // 0: nothing has been waited for

  // the word once it is `there`, or what it is when the time is over
  template <class Load, class There, class Clock, class Pause>
  SRQ_ANYWHERE uint32_t word(Load load, There there, Clock now, Pause pause) {
    uint32_t w = load();
    if (there(w)) return w;
    if (until == 0) until = now() + ticks;
    while (now() < until) {
      pause();
      w = load();
      if (there(w)) break;
    }
    return w;
  }
};

// How long that is, in ticks of 10 ns: 200 us, or what a text asks for, a decimal number of at most 10 ms.  With zero everybody
// works out alone what is not there at the first look.
constexpr uint32_t kExchangeTicks = 20000, kMostExchangeTicks = 1000000;
inline uint32_t exchange_ticks(const char* text) {
  if (!text || !*text) return kExchangeTicks;
  uint32_t n = 0;
  for (; *text; ++text) {
    if (*text < '0' || *text > '9') return kExchangeTicks;
    n = 10 * n + (uint32_t)(*text - '0');
    if (n > kMostExchangeTicks) return kExchangeTicks;
  }
  return n;
}

}  // namespace srq

#endif  // SRQ_EXCHANGE_WAIT_H_
