/* For the tests, not part of the library's interface (include/gspmd.h): which kernel the bf16 Dots of the calling thread
 * take.  Several kernels compute the same products, and a rule on sizes chooses; a test that is about the edges of one of
 * them pins that one, or asks afterwards which one ran.  Per thread, so that no other thread's calls are affected.  A
 * pinned kernel is taken where its operands and order of summation allow, elsewhere the rule holds as ever. */
#ifndef GSPMD_TESTING_H_
#define GSPMD_TESTING_H_
#include <stdint.h>

#ifdef __cplusplus
extern "C" {
#endif

enum {
  GSPMD_TESTING_BY_RULE = -1,
  GSPMD_TESTING_SCALAR = 0,     /* dot_fallback_kernel (float32 operands: dot_f32_kernel, which has no alternative) */
  GSPMD_TESTING_MFMA = 1,       /* dot_mfma_kernel */
  GSPMD_TESTING_MID = 2,        /* dot_mid_kernel: what dot_mfma_kernel takes with direct loads; others where nothing is summed and K-major operands have a tile of rows, columns */
  GSPMD_TESTING_SPLIT = 3,      /* dot_split_kernel: no partial sums along a contracting mesh dimension */
  GSPMD_TESTING_PAIR = 5        /* dot_pair_kernel: what dot_mfma_kernel takes with direct loads, nothing summed, K-contiguous operands in whole chunks of eight or padded rows */
};

typedef struct {
  int32_t kernel;       /* GSPMD_TESTING_* */
  int32_t row_blocks;   /* dot_split_kernel: 1, 2 or 4; others 0 */
  int32_t one_launch;   /* sums along a contracting mesh dimension: 1 in one launch where the operands allow, 0 in two; -1 by rule */
  int32_t dry_run;      /* pin: 1: Dots go no further than their launches, so that host logic can be tested without a GPU */
  /* last only: bytes of launch tables at the start of the workspace (0: they travel as kernel arguments), and where in the workspace
   * the partial sums or counters and slots of a sum lie */
  int64_t table_bytes, sums_begin, sums_end;
  int32_t moved_back;   /* last only: problems whose last tile column is moved back (all members of a sum, or none) */
  int32_t col_blocks;   /* dot_split_kernel: 2 (with 1 or 2 row blocks) or 4; pin: 0 is 4 */
} gspmd_testing_launch;

int32_t gspmd_testing_pin(const gspmd_testing_launch* pin);
int32_t gspmd_testing_last(gspmd_testing_launch* last);     /* of the thread's last Dot */

#ifdef __cplusplus
}
#endif
#endif /* GSPMD_TESTING_H_ */
