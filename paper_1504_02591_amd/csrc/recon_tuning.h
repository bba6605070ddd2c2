// Tuning knobs of the transform kernels, written by paper_1504_02591_amd/autotune.py (a -D on the
// compiler command line overrides them).  Tiles: packed z column pairs, y-pass columns, x-pass
// rows per block; middle radix split of the 512- and 1024-point transforms; z tiles per block of
// the z iteration.  The z and y knobs are timed at 128^3 and serve the sizes below 256 (the larger
// ones' tiles are fixed); RECON_TILE_X is timed at 512^3 and serves every size without its own.
// Chosen on a 128^3 correction pass of a batch of 16 (the values kept); ms per pass of each variant:
//   RECON_Z_TPB=1          0.5188
//   RECON_Z_TPB=2          0.5201
//   RECON_Z_TPB=4          0.5205
//   base                   0.5274
//   RECON_TILE_Z=8         0.5518
//   RECON_TILE_Y=8         0.7185
// Chosen on a 256^3 correction pass of a batch of 64 (the values kept); ms per pass of each variant:
//   base                   16.4111
//   RECON_TILE_X_256=4     16.5659
//   RECON_TILE_X_256=2     16.6420
// Chosen on a 512^3 correction pass (the values kept); ms per pass of each variant:
//   base                   2.1171
//   RECON_MID_512=2        2.1259
//   RECON_MID_512=1        2.1283
//   RECON_TILE_X=2         2.1399
//   RECON_TILE_X=8         2.1720
// Chosen on a 1024^3 correction pass (the values kept); ms per pass of each variant:
//   RECON_MID_1024=2       20.6981
//   RECON_MID_1024=1       20.8082
//   base                   20.9105
//   RECON_TILE_X_1024=4    21.4955
//   RECON_TILE_X_1024=8    22.3722
#pragma once
#ifndef RECON_TILE_Z
#define RECON_TILE_Z 16
#endif
#ifndef RECON_TILE_Y
#define RECON_TILE_Y 16
#endif
#ifndef RECON_Z_TPB
#define RECON_Z_TPB 8
#endif
#ifndef RECON_TILE_X
#define RECON_TILE_X 4
#endif
#ifndef RECON_MID_512
#define RECON_MID_512 0
#endif
#ifndef RECON_TILE_X_256
#define RECON_TILE_X_256 8
#endif
#ifndef RECON_TILE_X_1024
#define RECON_TILE_X_1024 2
#endif
#ifndef RECON_MID_1024
#define RECON_MID_1024 0
#endif
// Deposit launch shapes, timed on the 512^3 survey catalogues (ms per reconstruction, both catalogues):
//   brick accumulation threads per brick (accumulation)  256: 0.492   512: 0.440   1024: 0.507
//   binning blocks, one 128 KB LDS histogram each (count and scatter)  1024: 0.949   512: 0.856   256: 0.797
//   objects per loop trip (binning + accumulation + shift)
//     2: 0.811 + 0.456 + 1.138   4: 0.797 + 0.440 + 1.079   8: 0.811 + 0.460 + 1.087
//   reorder after the brick-order shift, chunks of one block (shift stage; a former build)
//     per_x apart: 1.096   adjacent (one trip per block), 2 / 4 / 8 chunks: 0.980 / 0.983 / 0.980
// Non-temporal hint on the transform passes' spectrum accesses (bit 0 stores, bit 1 loads), ms per
// correction pass with 0 / 1 / 2 / 3: 16 of 128^3 0.547 / 0.523 / 0.527 / 0.527, 64 of 256^3 16.97 / 16.72 /
// 16.84 / 16.41, 512^3 2.261 / 2.172 / 2.186 / 2.117, 1024^3 21.67 / 21.31 / 21.31 / 20.91 (Psi bit-identical).
// The same hint on the deposit's scattered brick-ordered copy made the binning 2.4x slower (0.79 -> 1.92 ms; a
// former build) and is not used.
// Binning above 512^3 (more bricks than one LDS histogram holds): per-block windows of the LDS histogram
// centred on the chunk's first object instead of global atomics for every object: count and scatter of 1.07e9
// lattice particles at 1024^3 179.9 -> 34.6 ms (a former build).
#ifndef RECON_X_WAVES
#define RECON_X_WAVES 0
#endif
#ifndef RECON_Z_DEFER
#define RECON_Z_DEFER 1
#endif
#ifndef RECON_BRICK_NT
#define RECON_BRICK_NT 512
#endif
#ifndef RECON_BIN_BLOCKS
#define RECON_BIN_BLOCKS 256
#endif
#ifndef RECON_OBJ_BATCH
#define RECON_OBJ_BATCH 4
#endif
#ifndef RECON_STREAM
#define RECON_STREAM 3
#endif
