// Host build of the device's sincos_near for the CPU tests.
#include "rr_device.h"

extern "C" {
void probe_sincos_near_f(float x, float* s, float* c) { rr::sincos_near(x, s, c); }
void probe_sincos_near_d(double x, double* s, double* c) { rr::sincos_near(x, s, c); }
}
