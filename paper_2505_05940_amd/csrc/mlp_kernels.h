// Jobs of the proposal network's kernel (mlp_kernels.hip), filled in by
// mlp_api.cpp.
#ifndef MLP_KERNELS_H
#define MLP_KERNELS_H

#include <hip/hip_runtime.h>

namespace modal {

// A product C[m, n] = sum_k A(m, k) B(n, k), or a matrix read from memory,
// and what is done with its tiles of 32 rows.  An operand of R rows by K is
// stored as ceil(R / 32) row blocks of kt >= ceil(K / 16) fragments of 512
// BF16: element (r, k) at 8 (64 (kt (r / 32) + k / 16) + r % 32 + 32 ((k % 16)
// / 8)) + k % 8.  Null pointers leave a part out.
struct MlpJob {
  int blocks;  // workgroups: mt ceil(N / width); 0: no such job
  int M, N;
  int width;   // of the tiles, 32 or 64
  int mt;      // ceil(M / 32)
  unsigned inv_mt;  // floor((2^32 - 1) / mt)
  int nk;                      // K in fragments of 16, in `slices` slices of ks
  int slices, ks;
  int akt, bkt, mkt, o1kt, o2kt;
  int vec;                     // src, C, p, m, v rows are whole aligned groups of four floats
  int relu;
  const unsigned short *A, *B;
  const float* src;            // without A: the matrix [..][N], rows idx[m] or m
  const long long* idx;
  const float* bias;           // [N], added
  const unsigned short* mask;  // operand (m, n): 0x8000 clears the element
  float* C;                    // [M][N]
  const float* Z;              // squared error against rows zidx[m] of Z [..][N]: the
  const long long* zidx;       // element becomes its gradient
  float *p, *m, *v;            // Adam on [M][N]: the element becomes the new parameter
  unsigned short *o1, *o2;     // the tile as operand (m, n) and as operand (n, m)
  float* csum;                 // column sums of each row block [ceil(M / 32)][N]
  const float* bsum;           // n_bsum row blocks' column sums [n_bsum][M], whose
  int n_bsum;                  // sum is the gradient bg [M] of the bias bp
  float *bg, *bp, *bm, *bv;
};

constexpr int kMlpJobs = 4, kMlpSlices = 8, kMlpThreads = 512;
struct MlpPhase {
  float lr, c1, c2, b1, b2, eps;  // Adam; c1, c2: 1 - beta^t
  const float* sched;             // if set, lr = sched[0], c1 = sched[2 k + 1], c2 = sched[2 k + 2]
  int k;
  float inv;                      // 1 / (B d) of the squared error
  float* lpart;                   // squared errors of the workgroups of a job with Z
  int n_lpart;
  float* loss;                    // += inv sum(lpart[0 .. n_lpart)), of an earlier launch
  MlpJob job[kMlpJobs];
};

hipError_t launch_mlp_phase(const MlpPhase& P, hipStream_t s);

}  // namespace modal
#endif
