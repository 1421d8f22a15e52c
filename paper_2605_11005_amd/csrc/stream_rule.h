// Which weights the experts' forward loads nontemporally.
//
// Weights that a call reads once and that do not stay in the Infinity Cache (256 MB) until the next call are: such loads leave the
// cache alone, and memory then delivers up to 13 % more (strips of 128 bytes of 1.9 GB: 6.3 -> 7.1 TB/s).  While the weights of the
// experts that have rows fit, a call made again finds them there; and what several tiles read, the later ones find there.  Up and down projection,
// us, loads as usual / nontemporal:
//   2.8 GB of weights   d = 7168, f = 2048, 32 experts of one row   326 + 167 / 291 + 153     of 128 rows by 1/r  329 + 169 / 300 + 155
//   604 MB              4096, 1536, 16 of 16 rows                   88 + 42 / 79 + 39
//   796 MB              2880, 2880, 16 of 16 rows                   97 + 57 / 84 + 52
//   302 MB              4096, 1536, 8 of 16 rows                    46 + 22 / 44 + 21
//   151 MB, again       4096, 1536, 4 of 16 rows                    29 + 14 / 39 + 16
//   138 MB, again       2048, 1408, 8 of 100 rows, two tiles each   57.5 (both) / 67.6        the same, other weights in between  64.2 / 68.8
//   151 MB, again       2048, 768, 16 of 65 rows, two tiles each    54.0 / 66.6               the same, other weights in between  61.7 / 67.6
// The line at what fits serves the layer that is called again with little in between.  Of weights that have not been read since, as a
// model of several layers finds them, nontemporal loads of one tile's are as fast or faster below it too: 22 + 16 / 21 + 15 at 138 MB.
#pragma once

// experts of w1, w3 and w2 in bf16 that fit
constexpr int cached_experts(int d, int f) { return (int)((256ll << 20) / (6ll * d * f)); }

// active: experts that have rows; cached: cached_experts; rows: of the expert whose weights are loaded; tile: rows of a tile
constexpr bool stream_weights(int active, int cached, int rows, int tile) { return active > cached && rows <= tile; }
