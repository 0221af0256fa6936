// LDS bytes of one wave's decode, as the kernels lay it out (carve_lds, carve_lds_n) and the
// host sizes its launches.
#ifndef FFS_LDS_SIZES_H
#define FFS_LDS_SIZES_H
#include <cstddef>
#include <cstdint>

namespace ffs_lds {

constexpr int kWave = 64;
constexpr size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Words of one row-ring buffer: a chunk of kWave / o_s ops of o_s words each,
// plus the record the op loop prefetches one past the chunk (read, never used).
constexpr int kRing = kWave + 16;

// LDS bytes before the profile region, and in all (cap = 0: no on-chip profile,
// the region still holds the genes).
constexpr size_t lds_head(int n) {
  return align_up((size_t)4 * n + 4, 16) + 2 * align_up((size_t)2 * n + 4, 16) + 4 * kRing;
}
constexpr size_t lds_bytes(int n, int cap) {
  const size_t prof = cap > 0 ? align_up(cap, 16) + kWave : 0, gene = align_up((size_t)4 * n, 16);
  return lds_head(n) + (prof > gene ? prof : gene);
}

// The chip form (LdsN), with room for the wide form of an off-chip redo.
constexpr int kChipSlots = 32768;
constexpr int kChipChunk = 16;  // ops whose rows are staged at once
constexpr size_t lds_head_n(int n, int omp) {
  return 3 * align_up((size_t)2 * n + 4, 16) + 4 * kChipChunk * omp;
}
constexpr size_t lds_bytes_n(int n, int omp, int cap) {
  const size_t prof = (size_t)3 * kWave + cap, gene = align_up((size_t)4 * n, 16);
  const size_t chip = lds_head_n(n, omp) + (prof > gene ? prof : gene);
  const size_t redo = lds_head(n) + gene;
  return chip > redo ? chip : redo;
}

// Whether decode_chip takes a decode: the default rules, and times past the slots
// still apart from the free time of a lane without a machine.
constexpr bool chip_rules(int rules, int cap) { return rules == 0 && cap <= kChipSlots; }

// LDS of a decode of n genes and rows of omp words under the decode rules `rules`.
constexpr size_t lds_bytes_rules(int rules, int n, int omp, int cap) {
  return chip_rules(rules, cap) ? lds_bytes_n(n, omp, cap) : lds_bytes(n, cap);
}

// Row width of the packed table.
constexpr int omp_of(int om) { return om <= 4 ? 4 : om <= 8 ? 8 : 16; }

// Waves of `bytes` of LDS each that a compute unit holds: at most 32, and its LDS (`lds` bytes)
// is given out in pieces of 1280 bytes.
constexpr int64_t waves_held(size_t bytes, int64_t lds) {
  const int64_t w = lds / (int64_t)align_up(bytes, 1280);
  return w < 32 ? w : 32;
}

// On-chip slots of pop decodes whose caller leaves them to the library: base (what the
// workspace is laid out for), or as many more as leave each of `cus` compute units room for as
// many waves as it holds at base and the population can use. With `groups`, the launches of
// island groups, one wave a unit is left over: they do not spread evenly (37 islands of 110
// decodes, 50 jobs, on exactly the 16 waves a unit that they need: 97.7 us a generation; at
// 4096 slots, 93.4). Less than half of base more is not taken unless no schedule can be longer:
// a schedule that outgrows both is found out later (8192 decodes of 130 jobs, 8 stages and 2
// machines under the power-aware rule: 4.65 ms a generation at 4928 slots, 4.34 at 4096). Past
// kChipSlots the decoder would be the general one. bytes(cap): LDS of one decode.
template <class F>
int roomy_slots(int base, int64_t horizon, int64_t pop, bool groups, int64_t cus, int64_t lds,
                F bytes) {
  if (base >= horizon || cus < 1) return base;
  const int64_t held = waves_held(bytes(base), lds);
  int64_t waves = (pop + cus - 1) / cus + groups;
  if (waves > held) waves = held;
  if (waves < 1) return base;
  const int64_t room = lds / waves / 1280 * 1280, h = (int64_t)align_up((size_t)horizon, 64);
  int64_t cap = (room - (int64_t)bytes(base) + base) / 64 * 64;
  if (cap > kChipSlots) cap = kChipSlots;
  if (cap > h) cap = h;
  return 2 * cap >= 3 * (int64_t)base || (cap >= h && cap > base) ? (int)cap : base;
}

// LDS of the decodes of a batch's size class of `cap` slots: room for the layouts of both kinds
// of decode rules, each at the most slots it runs with. A slot whose horizon needs fewer slots
// than its class takes the chip form also in a class past kChipSlots.
constexpr size_t batch_lds(int max_genes, int omp, int cap) {
  const size_t wide = lds_bytes(max_genes, cap);
  const size_t chip = lds_bytes_n(max_genes, omp, cap < kChipSlots ? cap : kChipSlots);
  return wide > chip ? wide : chip;
}

}  // namespace ffs_lds
#endif
