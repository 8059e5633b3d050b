// Lines between kernel forms that neither det_gemm_tile() nor det_qgemm_tile() shows.  The code takes them from here and
// det_fingerprint() states them from here, so that a receipt names the forms a build really has; why each lies where it does is
// said where it is used.
#pragma once

#define DET_QGEMM_FEW_ROWS 4       // rows of qgemm_few.hip, and of a norm inside 128-column packings
#define DET_QGEMM_NORM_ROWS 3      // rows that qgemm_few.hip normalizes itself
#define DET_QGEMM_MID16_ROWS 48    // rows of a tile of qgemm_mid.hip, 16-column packings
#define DET_QGEMM_MID32_ROWS 32    // and 32-column ones
#define DET_ATTN_NAMED_ROWS 16     // rows that name their slots go eight to a workgroup from here on
#define DET_ATTN_WALK_WGS 256      // and walk their chunks in launches of as many workgroups
#define DET_ATTN_FEW_PAIRS 16      // pairs of a group that does not walk there
#define DET_ATTN_TURN_CHUNKS 32    // chunks of a cache up to which they change places from stream to stream
