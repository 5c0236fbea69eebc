// Index map of the convolutional opening layer's gradient (k_open_grad_conv): where a
// thread's pixels lie. Plain C++ (constexpr functions run on the host and on the
// device), so that a host program can evaluate every index that the kernel forms.
#pragma once

namespace lp {
namespace open_conv {

constexpr int GNT = 1024;             // threads of the workgroup
constexpr int OCP = 8;                // pixels per thread and group of images
constexpr int OC_LDS = 12 * 1024;     // floats of the group's images with their zero halos

struct Group {
  int P, PW, PH;  // pixels of an image, padded row length, padded image
  int IM;         // images per group
};
constexpr Group group(int H, int W) {
  const int P = H * W, PH = (H + 2) * (W + 2);
  const int a = OCP * GNT / P, b = OC_LDS / PH;
  return {P, W + 2, PH, a < b ? a : b};
}

// Pixel i of a group (thread t holds i = t, t + GNT, ..): its image, the corner of its
// 3x3 window in the haloed images, and its offset in lam0 for channel co of C. Pixels
// beyond the group's IM images belong to no image: nothing may be stored for them.
struct Pixel {
  int im, at, gl;
};
constexpr Pixel pixel(const Group& g, int W, int C, int co, int i) {
  const int im = i / g.P, p = i - im * g.P, y = p / W;
  return {im, im * g.PH + y * g.PW + (p - y * W), (im * C + co) * g.P + p};
}

// images that the group at example e0 < B has
constexpr int images(const Group& g, int B, int e0) { return B - e0 < g.IM ? B - e0 : g.IM; }
// a pixel of an image that the group has: its values are read and counted
constexpr bool live(const Pixel& p, int n) { return p.im < n; }
// a pixel with a place in the haloed images (past the batch a zero is stored)
constexpr bool stored(const Group& g, const Pixel& p) { return p.im < g.IM; }
constexpr int store_index(const Group& g, const Pixel& p) { return p.at + g.PW + 1; }

}  // namespace open_conv
}  // namespace lp
