// Launchers private to the convolution translation units.
#pragma once
#include "anr_kernels.h"

namespace anr {

hipError_t launch_conv2d_direct(const ConvArgs& a, hipStream_t stream);
hipError_t launch_dwconv_direct(const ConvArgs& a, hipStream_t stream);

// Implicit-GEMM MFMA convolution.  Returns false in *taken when the geometry is
// outside what the kernel supports or the route rules it out (the caller then uses the
// general kernel).
hipError_t launch_conv2d_igemm(const ConvArgs& a, hipStream_t stream, bool* taken);

// Whether launch_conv2d_igemm would take the problem (same selection, nothing launched).
bool conv2d_igemm_takes(const ConvArgs& a);

// General implicit-GEMM convolution with gathered operands and optional split-K over a
// workspace.  *taken false: extents beyond its 32-bit offsets (the direct kernel runs then).
// *ws_fault as in launch_conv2d.
hipError_t launch_conv2d_gather(const ConvArgs& a, hipStream_t stream, bool* taken, int* ws_fault);
size_t conv2d_gather_workspace_bytes(const ConvArgs& a);
// Its estimated time for a 3 x 3 layer in microseconds (conv_taps_kernel, or conv_gather_kernel where the weights are not
// 16-byte aligned) and the bytes of its workspace; infinite where it does not take the call.
double conv2d_gather_estimate_us(const ConvArgs& a, size_t* workspace = nullptr);

// Estimated time of the kernel that the library's choice of a.route runs without a workspace for pieces, in microseconds;
// zero where that choice is to stand, the bytes of that kernel's workspace (conv2d_workspace_bytes of any layer that is
// not pointwise) and the order of a pack.  Pointers are taken as aligned and absent.
struct PackOrder {
    int tile, channels;      // of a pack that a patch kernel reads: output channels per tile, input channels per chunk, rows of a
                             // chunk's weights four floats apart; zero where the pack is a plain copy
};
double conv2d_estimate_us(const ConvArgs& a, size_t* workspace, PackOrder* pack);

// The general convolution on pieces made once per call (conv_pieces_kernel.h).  Bytes of workspace with which it runs, zero
// where another kernel is the faster one; *taken false: that, or a.ws is smaller or not aligned.  Always more than
// conv2d_workspace_bytes, so that a call which is given exactly those runs the kernel that needs them.
size_t conv2d_pieces_workspace_bytes(const ConvArgs& a);
hipError_t launch_conv2d_pieces(const ConvArgs& a, hipStream_t stream, bool* taken);

// Streaming kernel for pointwise layers with few channels (conv_pointwise_kernel.h); same contract.
hipError_t launch_conv2d_pointwise(const ConvArgs& a, hipStream_t stream, bool* taken);

// What a launch would do, for introspection (nothing is launched).
struct ConvRoute {
    int kernel;          // 1 patch-staging, 2 taps, 3 bigtaps, 4 gather, 5 direct, 6 pointwise stream (the public ANR_CONV_KERNEL_* values)
    int tile_m, tile_n, ksplit, wave_groups, work_groups;
    size_t workspace_bytes;
};
// Pointwise layers as a batched GEMM, weights times image, on planes that are no whole 16-byte units; same contract.
hipError_t launch_conv2d_pointwise_gemm(const ConvArgs& a, hipStream_t stream, bool* taken);
bool describe_conv2d_pointwise_gemm(const ConvArgs& a, ConvRoute* r);

// Kernel for images of two or three channels with 7 x 7 kernels (conv_stem.hip); same contract.
hipError_t launch_conv2d_stem(const ConvArgs& a, hipStream_t stream, bool* taken);

bool describe_conv2d_igemm(const ConvArgs& a, ConvRoute* r);
bool describe_conv2d_gather(const ConvArgs& a, ConvRoute* r);
bool describe_conv2d_pointwise(const ConvArgs& a, ConvRoute* r);
bool describe_conv2d_stem(const ConvArgs& a, ConvRoute* r);
void describe_conv2d(const ConvArgs& a, ConvRoute* r);

// Register-sliding 3x3 / stride 1 / pad 1 depthwise kernel; same contract.
hipError_t launch_dwconv3x3(const ConvArgs& a, hipStream_t stream, bool* taken);

}  // namespace anr
