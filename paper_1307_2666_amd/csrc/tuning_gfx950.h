// Built-in launch shapes for gfx950 (MI355X): the table hif_tuning_get
// returns until hif_tuning_set replaces it.  Written by
// paper_1307_2666_amd/tune.py from timings on one MI355X; see that script for
// the candidates and the problem sizes of each bucket.
//
// Medians (ms):
//   ID, 4096 problems of 33-64 columns: 4 waves 0.846, 8 waves 0.909, 16 waves 1.028
//   ID, 2048 problems of 97-128 columns: 4 waves 2.986, 8 waves 2.333, 16 waves 2.740
//   ID, 1024 problems of 161-192 columns: 8 waves 4.296, 16 waves 3.365
//   LU, 256 blocks of 257-512 rows: 256 threads 1.530, 512 threads 1.553, 1024 threads 1.735
//   LU, 64 blocks of 513-1024 rows: 512 threads 2.863, 1024 threads 3.238
//   8-RHS solve of a 384 x 384 factorization: 64 threads 1.463, 128 threads 1.361, 256 threads 1.318
#pragma once

// waves per problem of the register-resident pivoted QR, problems of at most
// 64, 128 and 192 columns
#define HIF_TUNED_ID_REG_WAVES {4, 8, 16}
// threads of the register-resident LU panel, panels of at most 512 and 1024 rows
#define HIF_TUNED_LU_PANEL_THREADS {256, 512}
// no effect: the row compression's trailing update has one shape
#define HIF_TUNED_ROWQR_UPDATE_WAVES 8
#define HIF_TUNED_ROWQR_UPDATE_KIND 1
// threads per record of the sweeps on sub-levels of at least 1024 records
#define HIF_TUNED_SWEEP_MANY_THREADS 256
