// Places of a chunk's waves in the order of the factorised sweeps (host and
// device).
//
// A chunk of the free list is ordered so that as many waves as there are one-cell
// nodes for hold nothing else.  The other waves take longer: they run the general
// form, and their nodes lie scattered over the chunk.  They are spread evenly
// among the chunk's waves, at other places in every chunk.  Consecutive workgroups
// go to the compute units in turn, so that with these waves at the chunks' ends
// the same few units of each XCD ran all of them: three problems of 10, 17 and 26
// nodes a side in 2149 workgroups, about one load of the chip, 22.1 us a sweep
// so and 16.9 spread (20.2 with the general form alone); 32^4, 17 controls: 28.3 and
// 24.8; 96^3 x 64, where the units balance by themselves, 17 controls 926 and 907,
// scan 64 + golden 12 1606 and 1626.
#pragma once

#ifdef __HIP__
#define DPO_HOST_DEVICE __host__ __device__
#else
#define DPO_HOST_DEVICE
#endif

namespace dpo {

constexpr int kOrderChunk = 4096;  // entries of the free list ordered together (64 waves of 64)

// slot[w]: place of the w-th wave of the chunk's n entries, of which the first
// `ones` are one-cell nodes and the rest are not.  Returns the bit of every place
// whose wave holds one-cell nodes alone.  A last, short wave keeps its place.
DPO_HOST_DEVICE inline unsigned long long place_waves(int n, int ones, int chunk, int* slot) {
  const int full = n / 64, pure = ones / 64 < full ? ones / 64 : full, mixed = full - pure;
  const int phase = (chunk * 39) & 63;  // about the golden section of the chunk's number
  // the m-th mixed wave at (m + phase / 64) full / mixed
  auto place = [&](int m) { return m < mixed ? (64 * m + phase) * full / (64 * mixed) : full; };
  unsigned long long bits = 0;
  int p = 0, m = 0, next = place(0);
  for (int s = 0; s < full; s++) {
    if (s == next) {
      slot[pure + m++] = s;
      next = place(m);
    } else {
      slot[p++] = s;
      bits |= 1ull << s;
    }
  }
  if (64 * full < n) {
    slot[full] = full;
    if (ones == n) bits |= 1ull << full;
  }
  return bits;
}

}  // namespace dpo
