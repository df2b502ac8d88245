// Launch-time constants of the built kernels, for the choice among them (estimate_seconds in ucl_api.hip).
//
// Each row was fitted to the launch times of its kernel on 80 to 1500 problems of random size (1..8192 rows and columns, K
// 64..16384; groups of 0..2000 rows; convolutions of 7..60 pixels a side, 32..512 channels; one MI355X, replays of a graph
// that walks three sets of buffers), kernels near the fastest of their problem weighing most.  Over those problems the
// kernel chosen by these rows is 0.2 to 1 % behind the fastest built one in the geometric mean (7 % at the 95th percentile
// at most).  The model before, one rate per tile size and a fixed cost, was 28 % behind for operands contiguous along
// K (it could not price the few-row kernels) and 3 to 9 % elsewhere.
//
//   fixed, round  microseconds of a launch and of every round of resident workgroups
//   gbs, tflops   what a CU copies into LDS (GB/s) and multiplies (TFLOP/s) with the kernel
//   step          microseconds a workgroup's chain needs per k-tile, copies and multiplications aside
//   out, hidden   weight of the output's bytes at 4.6 TB/s, and the share of that time that overlaps the loop
//   factor        correction of the whole, chosen for the choices it leads to rather than for the times
//   resident      workgroups per CU that the fit was made with
#pragma once

namespace ucl {

struct CostRow {
    short mode, la, lb, eight_bit;
    short tile_m, tile_n, tile_k, stages, k_groups, patch_c, resident;
    float fixed, round, gbs, tflops, step, out, hidden, factor;
};

static const CostRow kCostRows[] = {
    // mode la lb 8bit   tile            k-groups patch resident   fixed round  gbs  tflops step  out  hidden factor
    {0, 0, 0, 0,  256, 256, 64, 2,  1,   0, 1,  6.20f, 12.00f, 53.9f, 20.00f, 0.800f, 0.15f, 1.00f, 0.985f},
    {0, 0, 0, 0,  256, 256, 32, 4,  1,   0, 1,  5.99f, 12.00f, 51.6f, 19.96f, 0.391f, 0.17f, 0.97f, 1.000f},
    {0, 0, 0, 0,  256, 256, 32, 5,  1,   0, 1,  7.11f, 10.52f, 60.8f, 20.00f, 0.426f, 0.49f, 0.00f, 1.051f},
    {0, 0, 0, 0,  256, 128, 64, 2,  1,   0, 1,  4.55f, 6.09f, 57.1f, 20.00f, 0.628f, 0.52f, 0.01f, 1.000f},
    {0, 0, 0, 0,  256, 128, 32, 3,  1,   0, 2,  4.26f, 6.04f, 50.1f, 20.00f, 0.497f, 0.65f, 0.38f, 1.000f},
    {0, 0, 0, 0,  256, 128, 32, 4,  1,   0, 1,  3.67f, 7.47f, 50.2f, 19.74f, 0.253f, 0.22f, 1.00f, 1.000f},
    {0, 0, 0, 0,  128, 128, 64, 2,  1,   0, 2,  3.31f, 3.66f, 83.8f, 20.00f, 0.649f, 0.79f, 0.18f, 1.000f},
    {0, 0, 0, 0,  128, 128, 64, 3,  1,   0, 1,  3.41f, 3.95f, 47.4f, 20.00f, 0.483f, 0.51f, 0.75f, 0.985f},
    {0, 0, 0, 0,  128, 128, 32, 3,  1,   0, 3,  5.17f, 1.52f, 57.8f, 20.00f, 0.389f, 1.07f, 0.37f, 0.951f},
    {0, 0, 0, 0,  128, 128, 32, 4,  1,   0, 2,  4.19f, 2.97f, 55.8f, 20.00f, 0.221f, 0.84f, 0.40f, 1.030f},
    {0, 0, 0, 0,   64,  64, 64, 4,  1,   0, 2,  3.69f, 0.93f, 76.3f, 20.00f, 0.210f, 1.74f, 0.14f, 1.046f},
    {0, 0, 0, 0,   64,  64, 64, 4,  2,   0, 1,  2.39f, 2.88f, 62.5f, 20.00f, 0.108f, 0.94f, 0.02f, 1.000f},
    {0, 0, 0, 0,   64,  64, 32, 3,  1,   0, 4,  4.16f, 0.00f, 58.3f, 20.00f, 0.270f, 1.64f, 0.39f, 0.966f},
    {0, 0, 0, 0,   64,  64, 32, 4,  1,   0, 4,  4.20f, 0.00f, 60.2f, 20.00f, 0.179f, 1.74f, 0.30f, 0.966f},
    {0, 0, 0, 0,   64,  64, 64, 1,  8,   0, 1,  2.60f, 3.11f, 72.2f, 20.00f, 0.000f, 1.51f, 0.00f, 0.926f},
    {0, 0, 0, 0,   32,  64, 64, 1,  4,   0, 1,  2.18f, 3.07f, 80.3f, 20.00f, 0.004f, 1.83f, 0.01f, 0.985f},
    {0, 0, 0, 0,   32,  32, 64, 1,  4,   0, 1,  2.10f, 2.80f, 79.1f, 20.00f, 0.000f, 2.50f, 0.00f, 1.015f},
    {0, 0, 0, 0,   16,  32, 64, 1,  4,   0, 1,  1.90f, 2.62f, 91.2f, 20.00f, 0.000f, 0.73f, 0.03f, 1.000f},
    {0, 0, 0, 0,   16,  16, 64, 1,  4,   0, 2,  2.17f, 2.22f, 96.6f, 1.37f, 0.000f, 2.50f, 0.00f, 1.015f},
    {0, 0, 0, 1,  256, 256, 64, 2,  1,   0, 1,  6.83f, 11.56f, 68.6f, 20.00f, 0.784f, 0.49f, 0.03f, 1.000f},
    {0, 0, 0, 1,  256, 128, 32, 3,  1,   0, 2,  7.07f, 2.41f, 54.0f, 20.00f, 0.676f, 1.33f, 0.01f, 1.046f},
    {0, 0, 0, 1,  128, 128, 64, 2,  1,   0, 2,  5.02f, 1.64f, 97.1f, 20.00f, 0.545f, 1.57f, 0.00f, 0.985f},
    {0, 0, 0, 1,   64,  64, 64, 4,  1,   0, 2,  3.56f, 1.17f, 84.2f, 20.00f, 0.222f, 2.50f, 0.14f, 1.015f},
    {0, 0, 0, 1,   64,  64, 64, 4,  2,   0, 1,  2.17f, 3.19f, 76.0f, 20.00f, 0.298f, 1.55f, 0.02f, 1.000f},
    {0, 0, 0, 1,   32,  64, 64, 1,  4,   0, 1,  2.06f, 3.19f, 95.1f, 20.00f, 0.409f, 2.50f, 0.00f, 0.995f},
    {0, 0, 0, 1,   32,  32, 64, 1,  4,   0, 1,  2.01f, 2.90f, 104.0f, 20.00f, 0.246f, 2.50f, 0.00f, 1.030f},
    {0, 0, 0, 1,   16,  32, 64, 1,  4,   0, 1,  1.94f, 2.43f, 112.4f, 20.00f, 0.189f, 2.50f, 0.00f, 1.000f},
    {0, 0, 0, 1,   16,  16, 64, 1,  4,   0, 2,  2.10f, 2.21f, 107.4f, 20.00f, 0.102f, 2.50f, 0.00f, 1.015f},
    {0, 0, 4, 0,  256, 256, 64, 2,  1,   0, 1,  7.94f, 6.81f, 68.8f, 20.00f, 1.022f, 0.97f, 0.00f, 0.975f},
    {0, 0, 4, 0,  256, 128, 32, 3,  1,   0, 2,  3.90f, 2.68f, 109.2f, 20.00f, 0.696f, 1.81f, 0.00f, 1.000f},
    {0, 0, 4, 0,  128, 128, 64, 2,  1,   0, 2,  4.70f, 1.05f, 93.6f, 20.00f, 0.678f, 1.51f, 0.00f, 0.985f},
    {0, 0, 4, 0,  128, 128, 32, 4,  1,   0, 2,  6.47f, 0.00f, 64.7f, 20.00f, 0.231f, 1.12f, 0.00f, 0.966f},
    {0, 0, 4, 0,   64,  64, 64, 4,  1,   0, 2,  4.48f, 0.15f, 72.2f, 5.44f, 0.217f, 2.46f, 0.01f, 1.015f},
    {0, 0, 4, 0,   64,  64, 64, 4,  2,   0, 1,  2.13f, 2.83f, 80.3f, 6.66f, 0.460f, 2.50f, 0.00f, 1.000f},
    {0, 0, 4, 0,   64,  64, 32, 3,  1,   0, 4,  3.86f, 0.00f, 69.3f, 4.78f, 0.283f, 2.17f, 0.00f, 1.051f},
    {0, 5, 0, 0,  256, 256, 64, 2,  1,   0, 1,  8.12f, 7.15f, 78.8f, 20.00f, 0.986f, 0.86f, 0.02f, 1.127f},
    {0, 5, 0, 0,  128, 128, 64, 2,  1,   0, 2,  3.35f, 2.85f, 92.8f, 20.00f, 0.680f, 1.14f, 0.00f, 1.030f},
    {0, 5, 0, 0,  128, 128, 32, 4,  1,   0, 2,  4.82f, 1.84f, 68.2f, 20.00f, 0.248f, 0.97f, 0.01f, 1.000f},
    {0, 5, 0, 0,   64,  64, 64, 4,  1,   0, 2,  3.90f, 0.63f, 76.8f, 5.91f, 0.242f, 2.17f, 0.00f, 1.000f},
    {0, 5, 0, 0,   64,  64, 32, 3,  1,   0, 4,  3.51f, 0.00f, 78.5f, 4.82f, 0.356f, 2.12f, 0.01f, 1.041f},
    {0, 5, 4, 0,  256, 256, 64, 2,  1,   0, 1,  8.29f, 6.43f, 88.9f, 20.00f, 1.024f, 0.83f, 0.54f, 1.000f},
    {0, 5, 4, 0,  128, 128, 64, 2,  1,   0, 2,  2.49f, 4.02f, 95.9f, 20.00f, 0.632f, 0.76f, 0.03f, 1.046f},
    {0, 5, 4, 0,  128, 128, 32, 4,  1,   0, 2,  7.20f, 0.00f, 77.7f, 20.00f, 0.196f, 0.93f, 0.50f, 1.015f},
    {0, 5, 4, 0,  128, 128, 32, 4,  2,   0, 1,  3.23f, 5.38f, 78.4f, 20.00f, 0.000f, 0.59f, 0.02f, 1.000f},
    {0, 5, 4, 0,   64,  64, 64, 4,  1,   0, 2,  4.62f, 0.00f, 69.4f, 4.72f, 0.230f, 2.50f, 0.36f, 1.000f},
    {0, 5, 4, 0,   64,  64, 64, 4,  2,   0, 1,  3.05f, 1.98f, 69.1f, 6.77f, 0.426f, 2.50f, 0.16f, 1.191f},
    {0, 5, 4, 0,   64,  64, 32, 3,  1,   0, 4,  3.51f, 0.00f, 135.5f, 15.02f, 0.378f, 1.83f, 0.00f, 1.015f},
    {1, 0, 0, 0,  256, 256, 64, 2,  1,   0, 1,  8.61f, 4.23f, 70.1f, 6.58f, 0.360f, 2.33f, 0.63f, 1.000f},
    {1, 0, 0, 0,  256, 256, 32, 4,  1,   0, 1,  8.88f, 4.16f, 87.1f, 6.63f, 0.076f, 1.33f, 0.06f, 1.015f},
    {1, 0, 0, 0,  256, 256, 32, 5,  1,   0, 1,  8.30f, 5.57f, 65.8f, 6.98f, 0.109f, 2.43f, 0.57f, 1.000f},
    {1, 0, 0, 0,  256, 128, 32, 3,  1,   0, 2,  8.00f, 0.00f, 160.0f, 4.99f, 0.526f, 2.50f, 0.64f, 1.046f},
    {1, 0, 0, 0,  256, 128, 32, 4,  1,   0, 1,  2.25f, 4.31f, 76.0f, 5.04f, 0.345f, 0.97f, 0.13f, 1.000f},
    {1, 0, 0, 0,  128, 128, 64, 2,  1,   0, 2,  2.02f, 2.55f, 160.0f, 5.33f, 0.708f, 1.03f, 0.11f, 1.000f},
    {1, 0, 0, 0,  128, 128, 64, 3,  1,   0, 1,  1.62f, 3.00f, 160.0f, 2.71f, 0.370f, 0.00f, 1.00f, 1.030f},
    {1, 0, 0, 0,   64,  64, 64, 4,  1,   0, 2,  1.44f, 2.04f, 160.0f, 2.83f, 0.291f, 2.50f, 1.00f, 0.970f},
    {1, 0, 0, 0,   64,  64, 32, 3,  1,   0, 4,  3.43f, 0.25f, 160.0f, 2.17f, 0.275f, 1.39f, 0.00f, 1.083f},
    {1, 0, 0, 0,   32,  64, 64, 4,  4,   0, 3,  1.37f, 0.00f, 151.2f, 1.36f, 1.693f, 2.50f, 0.94f, 1.000f},
    {1, 0, 0, 0,   32,  32, 64, 4,  4,   0, 4,  2.23f, 0.00f, 62.2f, 20.00f, 0.581f, 0.00f, 1.00f, 1.000f},
    {1, 0, 0, 0,   32,  32, 64, 1,  4,   0, 1,  3.37f, 0.56f, 86.8f, 19.99f, 0.233f, 1.78f, 0.10f, 0.946f},
    {1, 0, 0, 1,  256, 256, 64, 2,  1,   0, 1,  1.00f, 10.30f, 160.0f, 20.00f, 1.437f, 2.50f, 0.00f, 1.000f},
    {1, 0, 0, 1,  128, 128, 64, 2,  1,   0, 2,  1.88f, 3.96f, 160.0f, 4.09f, 0.544f, 1.30f, 0.28f, 1.015f},
    {1, 0, 0, 1,   64,  64, 64, 4,  1,   0, 2,  2.18f, 2.21f, 47.3f, 20.00f, 0.216f, 0.00f, 1.00f, 1.000f},
    {1, 0, 0, 1,   32,  64, 64, 4,  4,   0, 3,  2.64f, 0.00f, 60.2f, 20.00f, 1.795f, 2.50f, 0.34f, 1.000f},
    {1, 0, 0, 1,   32,  32, 64, 4,  4,   0, 4,  2.82f, 0.00f, 57.1f, 20.00f, 1.115f, 2.48f, 0.01f, 1.000f},
    {1, 0, 0, 1,   32,  32, 64, 1,  4,   0, 1,  3.38f, 0.62f, 160.0f, 20.00f, 0.441f, 2.49f, 0.00f, 1.000f},
    {1, 0, 4, 0,  256, 256, 64, 2,  1,   0, 1,  6.77f, 5.86f, 66.3f, 6.07f, 0.247f, 0.88f, 0.07f, 0.937f},
    {1, 0, 4, 0,  128, 128, 32, 4,  1,   0, 2,  3.73f, 0.63f, 71.5f, 4.18f, 0.310f, 0.76f, 0.16f, 1.046f},
    {1, 0, 4, 0,   64,  64, 32, 3,  1,   0, 4,  2.75f, 0.00f, 160.0f, 1.95f, 0.495f, 0.00f, 1.00f, 1.133f},
    {2, 2, 0, 0,  256, 128, 64, 2,  1,   0, 1,  6.07f, 5.01f, 86.0f, 20.00f, 0.741f, 1.71f, 1.00f, 1.000f},
    {2, 2, 0, 0,  256, 128, 32, 3,  1,   0, 2,  6.07f, 3.87f, 65.0f, 20.00f, 0.546f, 0.00f, 1.00f, 1.000f},
    {2, 2, 0, 0,  256, 128, 32, 4,  1,   0, 1,  4.60f, 6.46f, 160.0f, 5.73f, 0.126f, 1.24f, 1.00f, 1.030f},
    {2, 2, 0, 0,  128, 128, 64, 2,  1,   0, 2,  7.24f, 0.73f, 82.8f, 20.00f, 0.493f, 2.50f, 0.85f, 0.970f},
    {2, 2, 0, 0,  128, 128, 64, 2,  2,   0, 1,  3.23f, 5.16f, 160.0f, 20.00f, 0.838f, 0.00f, 1.00f, 1.000f},
    {2, 2, 0, 0,  128, 128, 64, 3,  1,   0, 1,  3.24f, 5.10f, 70.9f, 20.00f, 0.418f, 1.61f, 0.64f, 1.000f},
    {2, 2, 0, 0,  128, 128, 32, 3,  1,   0, 3,  8.06f, 0.00f, 65.8f, 20.00f, 0.350f, 2.06f, 0.85f, 0.951f},
    {2, 2, 0, 0,  128, 128, 32, 4,  1,   0, 2,  5.60f, 2.84f, 67.9f, 20.00f, 0.200f, 2.25f, 1.00f, 1.000f},
    {2, 2, 0, 0,  128,  64, 64, 3,  2,   0, 1,  2.27f, 4.52f, 160.0f, 20.00f, 0.600f, 2.50f, 1.00f, 0.980f},
    {2, 2, 0, 0,   64,  64, 64, 4,  2,   0, 1,  2.56f, 3.73f, 160.0f, 20.00f, 0.324f, 1.45f, 0.71f, 0.951f},
    {2, 2, 0, 0,   64,  64, 32, 3,  1,   0, 4,  5.11f, 0.00f, 67.0f, 20.00f, 0.197f, 2.50f, 0.88f, 1.030f},
    {2, 2, 0, 0,   16,  32, 64, 1,  4,   0, 1,  2.07f, 5.23f, 160.0f, 20.00f, 0.278f, 2.50f, 0.00f, 1.000f},
    {2, 3, 0, 0,  256, 128, 32, 4,  1,  64, 1,  6.16f, 0.00f, 53.7f, 5.07f, 0.194f, 0.00f, 1.00f, 0.970f},
    {2, 3, 0, 0,  256, 128, 32, 4,  1, 128, 1,  1.00f, 0.00f, 160.0f, 3.67f, 0.371f, 0.00f, 1.00f, 1.191f},
    {2, 3, 0, 0,  128,  64, 32, 4,  1, 128, 3,  1.00f, 0.00f, 85.2f, 3.67f, 0.281f, 2.50f, 0.95f, 1.030f},
    {3, 2, 4, 0,  256, 128, 32, 3,  1,   0, 2,  6.61f, 2.85f, 160.0f, 20.00f, 0.865f, 2.27f, 1.00f, 1.000f},
    {3, 2, 4, 0,  128, 128, 32, 4,  1,   0, 2,  8.80f, 0.89f, 102.8f, 20.00f, 0.395f, 1.83f, 1.00f, 0.966f},
    {3, 2, 4, 0,  256,  64, 32, 4,  1,   0, 2,  4.29f, 5.06f, 160.0f, 4.58f, 0.500f, 0.00f, 1.00f, 1.156f},
    {3, 2, 4, 0,  128,  64, 32, 4,  1,   0, 3,  7.34f, 0.00f, 160.0f, 3.58f, 0.291f, 2.50f, 1.00f, 1.000f},
    {3, 2, 4, 0,   64,  64, 64, 4,  2,   0, 1,  3.47f, 4.91f, 160.0f, 20.00f, 0.561f, 0.00f, 0.00f, 0.937f},
    {3, 2, 4, 0,   64,  64, 32, 3,  1,   0, 4,  6.21f, 0.29f, 69.4f, 20.00f, 0.302f, 2.50f, 1.00f, 1.062f},
    {3, 3, 4, 0,  256, 128, 32, 4,  1,  64, 1,  5.78f, 0.00f, 160.0f, 4.39f, 0.397f, 0.00f, 1.00f, 0.831f},
    {3, 3, 4, 0,  256,  64, 32, 4,  1,  64, 2,  1.00f, 0.00f, 69.6f, 20.00f, 0.556f, 0.00f, 1.00f, 0.900f},
    {3, 3, 4, 0,  256,  64, 32, 4,  1, 128, 2,  1.00f, 0.00f, 73.0f, 3.30f, 0.344f, 0.00f, 1.00f, 1.116f},
    {3, 3, 4, 0,  128,  64, 32, 4,  1, 128, 3,  1.00f, 0.00f, 145.7f, 16.69f, 0.301f, 0.00f, 1.00f, 1.000f},
    {4, 5, 4, 0,  128, 128, 64, 2,  1,   0, 2,  8.29f, 2.55f, 58.9f, 5.08f, 1.176f, 0.00f, 0.00f, 1.000f},
    {4, 5, 4, 0,  128, 128, 32, 4,  1,   0, 2,  9.65f, 1.32f, 79.1f, 7.30f, 0.398f, 0.00f, 0.00f, 1.000f},
    {4, 5, 4, 0,   64,  64, 64, 4,  1,   0, 2,  7.47f, 2.13f, 85.9f, 16.48f, 0.499f, 0.00f, 0.00f, 1.000f},
    {4, 5, 4, 0,   64,  64, 32, 3,  1,   0, 4,  6.19f, 0.00f, 124.6f, 19.25f, 0.366f, 0.00f, 0.00f, 1.000f},
};

// Few-row kernels of four waves with more tiles than CUs, where they run with one stage buffer per wave (one_buffer() in ucl_api.hip; a CU then copies
// what its share of the tiles needs, whole rounds or not).  Fitted to 13000 problems of 1 to 3000 rows and up to 128 batches, 32 to 16384
// columns, K above 256 and up to 4096 (8-bit 8192); of 3200 others the kernel chosen is behind the fastest by 0.9 to 1.2 % (decoding, 1 to 300 rows), 1.4
// to 2.1 % (batches) and 1.2 % (more rows) in the geometric mean, with rows fitted to up to 300 rows and no batches, and those of the launches
// with several stages for the rest, 1.2 to 1.5, 10 to 13 and 3 to 4 %.  (The grouped kernels with one buffer have rows above, fitted to
// 9300 problems of 2 to 128 groups with 0 to 300 rows each: on 3100 others 0.4 to 1.5 % behind with 8-bit inputs, 1.0 to 2.4 % with 16-bit ones.)
static const CostRow kManyTilesRows[] = {
    {0, 0, 0, 0,   16,  16, 64, 1,  4,   0, 4,  3.17f, 0.00f, 95.1f, 20.00f, 0.525f, 2.25f, 0.01f, 1.117f},
    {0, 0, 0, 0,   16,  32, 64, 1,  4,   0, 4,  3.26f, 0.00f, 72.1f, 20.00f, 0.516f, 2.15f, 0.03f, 0.985f},
    {0, 0, 0, 0,   32,  32, 64, 1,  4,   0, 4,  3.21f, 0.10f, 78.9f, 20.00f, 0.485f, 2.36f, 0.01f, 1.000f},
    {0, 0, 0, 0,   32,  64, 64, 1,  4,   0, 3,  3.20f, 0.33f, 160.0f, 1.66f, 0.797f, 1.87f, 0.00f, 0.985f},
    {0, 0, 0, 1,   16,  16, 64, 1,  4,   0, 4,  3.49f, 0.00f, 73.0f, 20.00f, 0.418f, 2.50f, 0.36f, 1.080f},
    {0, 0, 0, 1,   16,  32, 64, 1,  4,   0, 4,  3.41f, 0.00f, 69.8f, 20.00f, 0.509f, 1.86f, 0.25f, 1.000f},
    {0, 0, 0, 1,   32,  32, 64, 1,  4,   0, 4,  3.01f, 0.60f, 73.4f, 20.00f, 0.490f, 1.30f, 0.04f, 1.000f},
    {0, 0, 0, 1,   32,  64, 64, 1,  4,   0, 3,  2.99f, 0.77f, 77.5f, 1.90f, 0.889f, 1.13f, 0.04f, 1.050f},
};

// Parallel split-K of the weight gradient: what the second launch costs with partial tiles of this kernel, microseconds and TB/s
// of partial tiles (fitted with the rows above: every built kernel with every power of two of slices, 440 geometries of up to
// 126000 pixels and 32 layers of a residual network at batches of 8 to 128).
struct SplitCostRow {
    short tile_m, tile_n, tile_k, stages;
    float fixed, tbs;
};
static const SplitCostRow kWgradSplitRows[] = {
    {128, 128, 32, 4,  0.00f, 3.33f},
    {128, 128, 64, 2,  0.00f, 3.62f},
    {64, 64, 32, 3,  1.28f, 2.19f},
    {64, 64, 64, 4,  0.00f, 2.41f},
};

// Tile kernels of 3x3 convolutions (forward at stride 1 and 2, data gradients at stride 1; rows of all that such a layer can get), for the choice between
// them and conv_held_kernel (tile_kernel_seconds).  kCostRows rank them among one another, but know neither the residual nor columns that
// fill no tile nor pixels of less than a line: 14 to 35 % off as times for the 128x128, 256x128 and 32-deep kernels, and the choice made with them
// took layers to conv_held_kernel that ran up to 1.6 times as fast here (17 x 56 x 56 x 128 -> 128 without a residual 21.8 us, there 33.3).
// Fitted to 79000 layers (1 to 64 images of 3 to 400 rows and 3 to 1024 columns, 8 to 1024 channels), 2 to 7 % off:
//   fixed, round, gbs, tflops, step   as in CostRow
//   out, residual, hidden             weight of the output's bytes at 4.6 TB/s, of the residual's, and the share that the loop hides
//   part, half_line                   what they take longer in a column of tiles that is not full, and where a row is not whole lines of 128 bytes
//   lines, few_n, stride2, odd_c      pixels copied beyond their bytes: whole lines where C < 64, filters of fewer than 64 columns, stride 2, C no multiple of 64
//   memory                            weight of the operands' trip from memory at 5.3 TB/s
struct ConvRow {
    short mode, tile_m, tile_n, tile_k, stages, k_groups, patch_c, resident;
    float fixed, round, gbs, tflops, step, out, residual, hidden, part, half_line, lines, few_n, stride2, odd_c, memory;
};
static const ConvRow kConvRows[] = {
    {2, 256, 128, 32, 3, 1,   0, 2,  6.24f, 2.31f, 175.4f, 7.76f, 0.786f,  0.66f, 0.84f, 0.00f, 0.49f, 0.91f,  0.71f, 30.00f, 1.45f, 0.00f, 1.32f},
    {2, 256, 128, 32, 4, 1,  64, 6,  2.33f, 1.12f, 62.6f, 5.59f, 0.597f,  0.42f, 0.83f, 0.03f, 0.71f, 1.70f,  0.68f, 6.40f, 0.00f, 0.00f, 4.55f},
    {2, 128, 128, 64, 2, 1,   0, 2,  4.75f, 1.31f, 178.6f, 8.77f, 0.665f,  1.18f, 1.13f, 0.02f, 0.53f, 0.41f,  0.00f, 7.16f, 0.68f, 1.41f, 1.31f},
    {2, 128, 128, 64, 2, 2,   0, 1,  4.10f, 3.72f, 124.9f, 4.84f, 0.007f,  0.65f, 1.03f, 0.08f, 0.80f, 1.24f,  0.00f, 3.03f, 0.87f, 1.45f, 1.67f},
    {2, 128, 128, 32, 3, 1,   0, 1,  4.95f, 0.05f, 276.0f, 30.00f, 0.239f,  1.04f, 1.19f, 0.00f, 0.22f, 0.48f,  3.00f, 19.12f, 2.53f, 0.57f, 1.51f},
    {2, 128,  64, 64, 3, 2,   0, 1,  3.64f, 2.17f, 173.0f, 2.96f, 0.008f,  1.27f, 1.53f, 0.03f, 0.16f, 0.94f,  0.00f, 1.46f, 1.68f, 1.16f, 1.88f},
    {2, 128,  64, 32, 4, 1, 128, 2,  4.80f, 0.00f, 242.1f, 5.40f, 0.146f,  1.98f, 1.37f, 0.03f, 1.20f, 0.22f,  1.14f, 6.37f, 0.00f, 0.00f, 0.00f},
    {2,  64,  64, 64, 4, 2,   0, 1,  4.58f, 1.64f, 135.8f, 30.00f, 0.251f,  0.85f, 2.05f, 0.02f, 0.05f, 0.57f,  0.46f, 1.47f, 0.32f, 0.43f, 0.82f},
    {2,  64,  64, 32, 3, 1,   0, 5,  5.24f, 0.39f, 333.9f, 2.59f, 0.138f,  0.99f, 0.84f, 0.03f, 0.00f, 0.28f,  3.00f, 5.50f, 0.00f, 0.00f, 1.72f},
    {2,  16,  32, 64, 1, 4,   0, 1,  5.26f, 1.98f, 166.5f, 30.00f, 0.177f,  4.62f, 6.51f, 0.07f, 0.00f, 0.00f,  0.00f, 0.00f, 0.20f, 0.00f, 0.01f},
    {3, 256, 128, 32, 4, 1,  64, 1,  6.82f, 6.77f, 900.0f, 30.00f, 0.000f,  0.32f, 0.71f, 0.00f, 0.72f, 1.46f,  2.29f, 0.30f, 0.00f, 0.00f, 1.60f},
    {3, 128, 128, 32, 4, 1,   0, 2,  6.44f, 5.44f, 277.8f, 4.97f, 0.000f,  0.71f, 0.82f, 0.00f, 0.69f, 0.41f,  1.79f, 17.65f, 1.37f, 3.00f, 4.08f},
    {3, 256,  64, 32, 4, 1,   0, 1,  5.25f, 3.01f, 301.5f, 4.54f, 0.337f,  0.18f, 0.79f, 0.00f, 0.00f, 0.89f,  1.78f, 0.47f, 1.04f, 3.00f, 7.95f},
    {3, 256,  64, 32, 4, 1,  64, 2,  6.74f, 0.00f, 581.0f, 4.65f, 0.246f,  0.40f, 1.26f, 0.00f, 0.09f, 1.90f,  1.43f, 30.00f, 0.00f, 0.00f, 2.38f},
    {3, 128,  64, 32, 4, 1,   0, 3,  7.41f, 0.00f, 222.3f, 3.77f, 0.265f,  1.76f, 0.81f, 0.02f, 0.00f, 0.41f,  1.87f, 8.03f, 1.05f, 1.21f, 3.51f},
    {3, 128,  64, 32, 4, 1, 128, 2,  5.14f, 1.07f, 900.0f, 4.87f, 0.144f,  1.11f, 1.25f, 0.04f, 0.11f, 0.71f,  1.97f, 24.53f, 0.00f, 0.00f, 2.65f},
    {3,  64,  64, 64, 4, 2,   0, 1,  2.64f, 6.27f, 82.7f, 30.00f, 0.393f,  1.34f, 2.17f, 0.01f, 0.27f, 0.26f,  0.65f, 1.05f, 2.93f, 0.08f, 3.03f},
    {3,  64,  64, 32, 3, 1,   0, 4,  5.91f, 0.95f, 64.7f, 2.66f, 0.231f,  0.33f, 0.66f, 0.06f, 0.05f, 1.15f,  1.18f, 1.00f, 0.27f, 0.00f, 6.19f},
};

// Launches of conv_held_kernel, microseconds (per byte; by wave groups over channels 1, 2, 4 and by waves that share a filter 1, 2, 4): fitted to 66000 launches
// of 12000 geometries (1 to 64 images of 5 to 80 pixels a side, 16 to 1024 channels), 7 % off; the plan chosen with them is 1.6 % behind the best of
// six measured ones on 12000 others.  On the 79000 layers of kConvRows, up to 1024 columns wide, the chosen plan's estimate is 6 % off, with the
// weights of the bytes that all move (the last three) fitted to them: 1 x 14 x 14 x 256 -> 1024 at stride 2 was priced 10.4 us and takes 7.4.
struct HeldCosts {
    double launch, pass[3], sharing[3], pair[3], next_pass;              // pair: a wave's two rows of 16 pixels
    double filter, filter_alone, pixels, pixels_alone;                   // bytes that a workgroup copies, by the share of busy CUs and by themselves
    double memory, moved, weights;                                       // bytes that all of them move
};
static const HeldCosts kHeldCosts = {2.933, {1.864, 2.100, 2.098}, {0.178, 0.389, 0.137}, {1.320, 1.482, 1.512}, 1.565,
                                     3.83e-6, 0.14e-6, 11.4e-6, 19.7e-6, 0.764, 0.283e-6, 0.317e-6};

}  // namespace ucl
