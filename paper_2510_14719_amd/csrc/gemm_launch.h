// Internal seam between the host-side C ABI (gemm_api.cpp) and the kernel (gemm_nt_kernel.hip).
#pragma once

struct GemmLaunchArgs {
    const void* a;   // [M][K]
    const void* b;   // [N][K]
    void* c;         // [M][N]
    int M, N, K;
    int dtype;       // 0 = fp16, 1 = bf16 (for the 8-bit product: the type of c; a and b are E4M3 bytes)
    void* stream;    // hipStream_t
    int config = 0;  // 0 = chosen by M, N and K, 1 ... 4 = a fixed configuration of gemm_nt_kernel.hip / gemm_nt_fp8_kernel.hip (waves per workgroup, paired copies)
};

// Enqueue the kernel for already-validated arguments.  0 on success, -1 if HIP refused the launch.
int gemm_launch(const GemmLaunchArgs& a);

// What configuration 0 takes; in_type 0 = fp16, 1 = bf16, 2 = E4M3 operands.
int gemm_default_launch(const GemmLaunchArgs& a, int in_type);
// The kernels it chooses from (gemm_nt_tile_kernel.hip): shape 0 (256 x 256 of C per workgroup), 1 (64 x 64), 2 or 3 (128 x 128).
int gemm_tile_launch(const GemmLaunchArgs& a, int in_type, int shape);
// The shape for rows of row_bytes (K elements).
int gemm_tile_shape(int M, int N, long long row_bytes);

// The smallest tiles of C (gemm_nt_narrow_kernel.hip), in the place of shape 1 where gemm_narrow_tile says 32 or 16 and not 0.
int gemm_narrow_tile(int M, int N, long long row_bytes, bool fp8);
int gemm_narrow_launch(const GemmLaunchArgs& a, int in_type, int tile);

// Rows of C per workgroup (0), columns (1), K tile (2), LDS stages (3), threads per workgroup (4).
int gemm_launch_tile_param(int which);

// The same two calls for the product of 8-bit-float (E4M3) operands (gemm_nt_fp8_kernel.hip).
int gemm_fp8_launch(const GemmLaunchArgs& a);
int gemm_fp8_launch_tile_param(int which);
