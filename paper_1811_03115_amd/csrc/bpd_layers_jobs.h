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
//   one slot per job, 8 jobs of 10 rows   500: 112 alone, 118 (two), 124 (three)   1000: 130, 132, 140   1150: 137, 139, 141   1300: 144, 140, 144   1500: 147, 142, 145   2000: 164, 154, 156   3000: 198, 174, 168
//   1 job of 10 rows                      600: 107, 114, 113   1000: 115, 116, 122   1150: 122, 122, 121   1300: 127, 122, 122   2000: 142, 129, 130   3000: 170, 143, 139
//   two slots, 8 jobs of 16 rows          500: 128   1000: 149   2000: 188   3000: 223 (two, measured with flags behind the results: 7 .. 14 more than alone)
// (by events.  They cross at 1150 .. 1300, by 3 % where the line is; 3072 positions, the longest caches measured, gain 30.)
constexpr int LK_SPLITS = 3;
inline int layers_split(int slots, long keys) { return keys > 1024 && layers_per_job(slots) == 1 ? LK_SPLITS : 1; }
// ... and of wide_layers_kernel: one block of at most 16 rows of four slots.  Keys held and positions of the source that was encoded (not what the context
// has room for): one workgroup has all of a head's, the chain of kernels deals them out, so that the two cross.  Six layers, us, chain and one kernel:
//   keys     1 slot x 10 rows   64: 185, 135   1000: 207, 160   1300: 222, 173   2000: 230, 190   3000: 230, 226        1 x 1   64: 183, 104   1000: 220, 129   1300: 221, 144   3000: 221, 199
//            4 x 4              64: 201, 141   1000: 235, 177   2000: 239, 216   3000: 254, 250        5 x 8   64: 253, 180   1000: 294, 218   3000: 321, 289
//            8 x 8              64: 259, 212   1000: 300, 260   3000: 360, 335        16 x 4   64: 263, 241   1000: 340, 332   1300: 353, 363   2000: 393, 408
//   source   1 x 10             32: 184, 134   1000: 212, 169   1300: 213, 178   2000: 215, 201        16 x 4  32: 277, 244   1000: 361, 344   1300: 381, 376   2000: 424, 441
// (by events around the launches: some 5 us too much each.)  1024 of either is where 16 x 4, the first to, nearly crosses in keys; the others gain 40 .. 90 us there, and cross
// at 3000 and beyond.
constexpr long WIDE_LAYERS_KEYS = 1024;
// tall_layers_kernel: more rows, of up to 16 slots
constexpr int TALL_LAYERS_ROWS = 64;
inline bool tall_layers_fit(int slots, int R, long keys, long src) { return slots <= 16 && R <= 16 && slots * R > 16 && slots * R <= TALL_LAYERS_ROWS && keys <= WIDE_LAYERS_KEYS && src <= WIDE_LAYERS_KEYS; }
inline bool wide_layers_fit(int slots, int R, long keys, long src) { return slots <= 4 && slots * R <= 16 && keys <= WIDE_LAYERS_KEYS && src <= WIDE_LAYERS_KEYS; }
