// Name of the kernel that a 16-bit (f16) 3x3 or 1x1 convolution launches, for shapes read from the command line as
// ksize,n,cin,cout,h,w,fp32_output,residual: what the tests at the edges of a tile need to know of a shape.  Host code only.
#include <cstdio>

#include "common.hpp"

int main(int argc, char** argv) {
  for (int i = 1; i < argc; ++i) {
    wmdec::ConvArgs a;
    int f32 = 0, res = 0;
    if (sscanf(argv[i], "%d,%d,%d,%d,%d,%d,%d,%d", &a.ksize, &a.n, &a.cin, &a.cout, &a.h, &a.w, &f32, &res) != 8) return 1;
    a.op_dtype = a.x_dtype = a.res_dtype = WMDEC_F16;
    a.y_dtype = f32 ? WMDEC_F32 : WMDEC_F16;
    if (res) a.res = &a;   // (that there is one)
    printf("%s\n", wmdec::conv_kernel_label(a));
  }
  return 0;
}
