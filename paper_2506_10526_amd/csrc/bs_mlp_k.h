// Argument blocks and launchers of the variance-surrogate MLP kernels.
#pragma once
#include <hip/hip_runtime.h>

constexpr int MLP_IN = 4, MLP_HID = 256;
constexpr int MLP_OFF_W1 = 0;
constexpr int MLP_OFF_B1 = MLP_OFF_W1 + MLP_HID * MLP_IN;    // 1024
constexpr int MLP_OFF_W2 = MLP_OFF_B1 + MLP_HID;             // 1280
constexpr int MLP_OFF_B2 = MLP_OFF_W2 + MLP_HID * MLP_HID;   // 66816
constexpr int MLP_OFF_W3 = MLP_OFF_B2 + MLP_HID;             // 67072
constexpr int MLP_OFF_B3 = MLP_OFF_W3 + MLP_HID * MLP_HID;   // 132608
constexpr int MLP_OFF_W4 = MLP_OFF_B3 + MLP_HID;             // 132864
constexpr int MLP_OFF_B4 = MLP_OFF_W4 + MLP_HID;             // 133120
constexpr int MLP_NPARAM = MLP_OFF_B4 + 1;                   // 133121
constexpr int MLP_NSTATE = MLP_NPARAM + 10;                  // + mu_x[4], s_x[4], mu_t, s_t

// The row-local part of the network (k_mlp_rows) and the partials of its gradient.
constexpr int MR_ROWS = 16;          // rows a block carries through the network at a time
constexpr int MR_MAX_BLOCKS = 1024;  // row blocks; larger batches loop
constexpr int MR_PART = 2048;        // per half block: dW1 [256][4], db1, db2, db3, dw4
constexpr int MLP_MAX_SPLITS = 8;    // row splits of the weight gradients
struct MlpRowArgs {
  const float* X;      // [n][4]: normalised (training) or raw (prediction)
  const float* t;      // training: normalised targets [n]
  const float* p;      // parameters
  const float* norm;   // prediction: mu_x[4], s_x[4], mu_t, s_t
  int n;
  float* y;            // prediction [n]
  float *H1, *H2, *dZ2, *dZ3;   // training: [n][256]
  float* vpart;        // [2 row blocks][MR_PART]
  float* wpart;        // [splits][2][256][256]
  double* lpart;       // [row blocks][2]: squared residuals, dy
};

// Device-resident training state read by the Adam kernel (so a captured step can be replayed).
struct TrainState {
  int step;     // Adam steps taken so far (bias correction uses step + 1)
  int local;    // steps taken in the current run (cosine schedule position)
  int K;        // steps of the current run
  int cosine;
  float lr, b1, b2, eps;
};

int mlp_row_blocks(int n);
void launch_mlp_predict(const MlpRowArgs& a, hipStream_t s);
void launch_mlp_loss_grad(const MlpRowArgs& a, float* grad, double* loss, hipStream_t s);
void launch_adam(float* p, const float* g, float* m, float* v, int n, const TrainState* ts, hipStream_t s);
void launch_train_set(TrainState* ts, float lr, int K, int cosine, int reset_step, hipStream_t s);
void launch_fit_norm(const float* X, const float* t, int n, float* norm, hipStream_t s);
void launch_normalise(const float* X, const float* t, int n, const float* norm, float* Xn, float* tn, hipStream_t s);
void launch_mlp_init(float* p, unsigned long long seed, hipStream_t s);
void launch_to_bf16(const float* x, void* y, int n, hipStream_t s);
void launch_bf16_forward(const float* Xn, int n, const float* p, const float* norm, const void* W2b, const void* W3b,
                         const void* w4b, void* H1, void* H2, float* y, hipStream_t s);
// Gaussian flag proxy: xi[s][nu] for s = 0..nsmax (device float64 [nsmax+1][nc]) and the cube
// V[nu][u][v] = a(nu) xi[q_u^2 + q_v^2][nu] on support cells (complex128 [nc][n][n/2+1]).
void launch_var_xi(int nc, int nsmax, double cperp2, double cpar2, double pk_index, double* xi, hipStream_t s);
void launch_var_cube(int n, int nh, int nc, int smax, const double* a, const double* xi, void* V, hipStream_t s);
