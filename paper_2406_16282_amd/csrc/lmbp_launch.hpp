// Internal launcher declarations between the C ABI layer and the kernel files.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace lmbp {

enum { kGelu = 0, kSilu = 1 };

constexpr int kXcds = 8;          // consecutive blocks go to them in turn
constexpr int kMaxDevices = 64;   // of one process

// The current device and its CU count (queried once per device).
hipError_t current_device(int& dev, int& cus);

// Runtime tables of a general family member (kernel argument, passed by value):
// thresholds t[0..2^k-2] as fp32 round-down values, levels lv[0..2^k-1] in fp32.
struct StepTable {
  float t[15];
  float lv[16];
};

hipError_t launch_act_fwd(int act, bool bf16, int64_t n, const void* x, void* y,
                          uint32_t* codes, bool vec_ok, hipStream_t s);
hipError_t launch_act_bwd(int act, bool bf16, int64_t n, const void* dy, const uint32_t* codes,
                          void* dx, bool vec_ok, hipStream_t s);

// Gated form h = act(g) * u (only act = kSilu is instantiated).
hipError_t launch_glu_fwd(int act, bool bf16, int64_t n, const void* g, const void* u, void* h,
                          void* s, uint32_t* codes, bool vec_ok, hipStream_t st);
hipError_t launch_glu_bwd(int act, bool bf16, int64_t n, const void* dh, const void* u,
                          const void* s, const uint32_t* codes, void* dg, void* du, bool vec_ok,
                          hipStream_t st);

// vec_ok: every tensor pointer 16-byte aligned and cols * element bytes a
// multiple of 16 (each row starts on a vector boundary).
hipError_t launch_norm_fwd(bool ln, bool bf16, int64_t rows, int64_t cols, float eps,
                           const void* x, void* z, float* rstd, bool vec_ok, hipStream_t s);
hipError_t launch_norm_bwd(bool ln, bool bf16, int64_t rows, int64_t cols, const void* dz,
                           const void* z, const float* rstd, void* dx, bool vec_ok,
                           hipStream_t s);

hipError_t launch_stepact_fwd(int act, int bits, bool bf16, int64_t n, const void* x, void* y,
                              uint32_t* codes, bool vec_ok, const StepTable& tab, hipStream_t s);
hipError_t launch_stepact_bwd(int bits, bool bf16, int64_t n, const void* dy, const uint32_t* codes,
                              void* dx, bool vec_ok, const StepTable& tab, hipStream_t s);

// z = bf16(x W^T + bias) (bf16 operands, fp32 accumulation); y = act(z), codes of z;
// z stored when non-null. N % 16 == 0, K % 8 == 0, x/w/y/z 16-byte aligned.
hipError_t launch_linear_act_fwd(int act, int64_t M, int64_t N, int64_t K, const void* x,
                                 const void* w, const void* bias, void* y, uint32_t* codes,
                                 void* z, hipStream_t s);

// Gated form: g = bf16(x Wg^T), u = bf16(x Wu^T); h = SiLU(g) * u, s = SiLU(g), u stored,
// codes of g; g stored when non-null. Same requirements as launch_linear_act_fwd.
hipError_t launch_linear_glu_fwd(int64_t M, int64_t N, int64_t K, const void* x, const void* w_gate,
                                 const void* w_up, void* h, void* s_out, void* u, uint32_t* codes,
                                 void* g, hipStream_t s);

// The same layers with MS-RMSNorm in front (Sec. 5.2 eq. norm_linear): x [M x K] is the
// norm's input. The norm kernel writes rstd (fp32, per row) and the norm's output z_norm
// [M x K]; the GEMM runs on x and scales each row's fp32 sums by its rstd before the
// bias. pre / g: the rounded pre-activation (gate), stored when non-null. x, w, z_norm
// 16-byte aligned; K % 8 == 0, N % 16 == 0.
hipError_t launch_linear_rms_act_fwd(int act, int64_t M, int64_t N, int64_t K, float eps,
                                     const void* x, const void* w, const void* bias, void* y,
                                     uint32_t* codes, void* pre, void* z_norm, float* rstd,
                                     hipStream_t s);
hipError_t launch_linear_rms_glu_fwd(int64_t M, int64_t N, int64_t K, float eps, const void* x,
                                     const void* w_gate, const void* w_up, void* h, void* s_out,
                                     void* u, uint32_t* codes, void* g, void* z_norm, float* rstd,
                                     hipStream_t s);

// The form that the fused forward of a layer runs in on the current device (256 CUs without
// one): 0, 1 split-K with 16, 32 rows; 2 .. 5 tiles of 256 x 256, 128 x 256, 128 x 128, 64 x
// 128; and the most tiles that a block computes.
struct LinearForm {
  int form;
  int64_t rounds;
};
LinearForm linear_form(bool gated, int64_t M, int64_t N, int64_t K);

// How dW is computed on the current device (256 CUs without one): made once per call, for K =
// 0 if dw is not asked for.
struct LinearGradPlan {
  int tile = 0;        // 0: 256 x 256, 1: 128 x 256, 2: 128 x 128
  int64_t splits = 1;  // shares of the rows that hold any
  int64_t per = 1;     // 64-row steps per share
};
LinearGradPlan linear_grad_plan(int64_t M, int64_t N, int64_t K);
size_t linear_grad_workspace(int64_t M, int64_t N, int64_t K, bool bias, const LinearGradPlan& plan);
// The tile of dW (0 .. 2: 256 x 256, 128 x 256, 128 x 128), the shares that its rows are split
// into, and the most units of work that a block takes.
struct LinearGradForm {
  int tile;
  int64_t splits, rounds;
};
LinearGradForm linear_grad_form(int64_t M, int64_t N, int64_t K);

// Backward of a fused linear layer's parameters. db non-null: dz = dy slope[code] is
// computed here (act) and db is the column sums of dz; else dz is an input. dw non-null:
// dw = bf16(dz^T x). Workspace of linear_grad_workspace bytes (same sizes and plan; bias: db
// non-null; K = 0 if dw is null). N % 16 == 0, K % 8 == 0, every tensor 16-byte aligned, db 2-byte
// aligned.
hipError_t launch_linear_grad(int act, int64_t M, int64_t N, int64_t K, const void* dy, const uint32_t* codes,
                              const void* x, void* dz, void* dw, void* db, void* workspace,
                              const LinearGradPlan& plan, hipStream_t s);

hipError_t launch_copy(const void* src, void* dst, int64_t bytes, hipStream_t s);

}  // namespace lmbp
