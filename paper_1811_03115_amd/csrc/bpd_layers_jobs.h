// How decoder blocks are dealt to the jobs of layers_kernel (bpd_layers.h), for the kernel and for the host.
#pragma once

constexpr int LK_PLACES = 32, LK_XCDS = 16, LK_JOBS = 8;
constexpr int LK_CTL = 32, LK_FLAGS = 64, LK_AREA = 192;        // words of an XCD's area: [0] registered; members, then jobs; flags [wave][member]
constexpr int LK_NEXT_JOB = LK_XCDS * LK_AREA, LK_WORDS = LK_NEXT_JOB + 32;
// Slots of a job: they are dealt evenly to at most LK_JOBS of them, and a job holds at most 16 rows of four slots
inline int layers_per_job(int slots) { return (slots + LK_JOBS - 1) / LK_JOBS; }
inline bool layers_fit(int slots, int R) { return layers_per_job(slots) <= LK_PLACES / 8 && layers_per_job(slots) * R <= 16; }
// Workgroups that share the self-attention of a (head, slot): sharing costs the next operator the merging of their results, and members that fetch weights
// meanwhile.  Six layers in us, by keys:
//   one slot per job, 8 jobs of 10 rows   500: 127 alone, 130 (two), 133 (three)   1000: 141, 142 (two), 144 (three)   1300: 153, 149 (three)   1500: 155, 150 (two, three), 156 (four)   3000: 220, 178 (three), 188 (two)
//   1 job of 10 rows                      600: 124, 130   1000: 133, 137   1300: 145, 140   3000: 188, 159
//   two slots, 8 jobs of 16 rows          500: 140, 154   1000: 158, 172   2000: 205, 212 (two)
constexpr int LK_SPLITS = 3;
inline int layers_split(int slots, long keys) { return keys > 1024 && layers_per_job(slots) == 1 ? LK_SPLITS : 1; }
// ... and of wide_layers_kernel: one block of at most 16 rows of four slots.  Keys held and positions of the source that was encoded (not what the context
// has room for): one workgroup has all of a head's, the chain of kernels deals them out, so that the two cross.  Six layers, us, chain and one kernel:
//   keys     1 slot x 10 rows   64: 188, 154   1000: 215, 188   1300: 225, 204   2000: 228, 225   3000: 248, 260        1 x 1   1000: 182, 152   1300: 182, 166
//            4 x 4              64: 211, 169   1000: 248, 207   2000: 251, 241   3000: 266, 277        5 x 8   64: 254, 189   1000: 294, 228   3000: 324, 296
//            8 x 8              1000: 303, 272   3000: 363, 348       16 x 4   64: 279, 260   1000: 347, 342   1300: 371, 372   2000: 409, 416
//   source   1 x 10             32: 185, 153   1000: 219, 186   1300: 232, 208   2000: 236, 241        16 x 4  1000: 361, 352   1300: 381, 385
// (by events around the launches: some 5 us too much each.)  1024 of either is where 16 x 4, the first to, nearly crosses; the others gain 20 .. 65 us there: blocks of up
// to 16 rows lose that by 1700 .. 2500, taller ones of up to eight slots beyond 3000.
constexpr long WIDE_LAYERS_KEYS = 1024;
// tall_layers_kernel: more rows, of up to 16 slots
constexpr int TALL_LAYERS_ROWS = 64;
inline bool tall_layers_fit(int slots, int R, long keys, long src) { return slots <= 16 && R <= 16 && slots * R > 16 && slots * R <= TALL_LAYERS_ROWS && keys <= WIDE_LAYERS_KEYS && src <= WIDE_LAYERS_KEYS; }
inline bool wide_layers_fit(int slots, int R, long keys, long src) { return slots <= 4 && slots * R <= 16 && keys <= WIDE_LAYERS_KEYS && src <= WIDE_LAYERS_KEYS; }
