// The generator's quotients and roots are a hardware estimate and one correction by fused multiply-adds.  For all 2^23
// uniforms: where would the result depend on an estimate's last bit?  Prints "dist word" for every uniform at which an estimate
// that is one unit in the last place off the correctly rounded one (v_rcp_f32 and v_rsq_f32 are that accurate)
// gives another result than the IEEE operators, and "general" if a correctly rounded estimate ever does.
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>

static float of_bits(uint32_t b) { float f; std::memcpy(&f, &b, 4); return f; }
static uint32_t bits(float f) { uint32_t b; std::memcpy(&b, &f, 4); return b; }
static float off_by(float f, int units) { return of_bits(bits(f) + (uint32_t)units); }

static float quotient(float t, float d, int units) {
  const float r = off_by((float)(1.0 / (double)d), units), q = t * r;
  return std::fmaf(std::fmaf(-d, q, t), r, q);
}
static float root(float a, float estimate_at, int units) {
  const float y = off_by((float)(1.0 / std::sqrt((double)estimate_at)), units);
  const float g = a * y, h = 0.5f * y;
  return std::fmaf(std::fmaf(-g, g, a), h, g);
}
// f * log(u) from the quotient s of its series
static float series(float s, int ne, float f) {
  const float w = s * s;
  float p = std::fmaf(w, 0.111111112f, 0.142857149f);
  p = std::fmaf(w, p, 0.2f);
  p = std::fmaf(w, p, 0.333333343f);
  p = std::fmaf(w, p, 1.0f);
  return std::fmaf((float)ne, -f * 0.693147182f, (2 * f * s) * p);
}
static float exponential(float y) {
  const int n = (int)(y * 1.44269502f + 0.5f);
  const float r = std::fmaf(-(float)n, 1.42860677e-6f, std::fmaf(-(float)n, 0.693145752f, y));
  float p = std::fmaf(r, 1.38888892e-3f, 8.33333377e-3f);
  p = std::fmaf(r, p, 4.16666679e-2f);
  p = std::fmaf(r, p, 0.166666672f);
  p = std::fmaf(r, p, 0.5f);
  p = std::fmaf(r, p, 1.0f);
  p = std::fmaf(r, p, 1.0f);
  return of_bits(bits(p) + ((uint32_t)n << 23));
}

int main() {
  for (uint32_t n = 0; n < (1u << 23); ++n) {
    const uint32_t b = bits((float)((n + 0.5) * 0x1p-23));
    const int ne = (int)(0x3F3504F4u + 0x7FFFFFu - b) >> 23;
    const float m = of_bits(((uint32_t)ne << 23) + b), t = m - 1.0f, d = m + 1.0f, s = t / d;
    const float normal = series(s, ne, -2.0f), student = 3.0f * (exponential(0.666666687f * series(s, ne, -1.0f)) - 1.0f);
    const float at = std::fmax(student, 1e-30f);
    for (int dist = 0; dist < 2; ++dist) {
      const float a = dist ? student : normal, e = dist ? at : normal;
      bool differs = false;
      for (int units = -1; units <= 1; ++units) {
        const bool here = bits(quotient(t, d, units)) != bits(s) || bits(root(a, e, units)) != bits(std::sqrt(a));
        if (units == 0 && here) std::printf("general %u\n", n);
        differs |= here;
      }
      if (differs) std::printf("%d %u\n", dist, n);
    }
  }
}
