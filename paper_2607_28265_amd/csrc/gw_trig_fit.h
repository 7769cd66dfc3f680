// Generated by gen_trig_fit.py; do not edit.
// sin(2 pi r) = r sum_k s[k] r^2k and cos(2 pi r) = sum_k c[k] r^2k, |r| <= 1/2
// (largest absolute errors 2.1e-11 and 1.2e-10).
#pragma once
namespace gw {
struct TrigFit {
  double s[8];
  double c[8];
};
inline TrigFit make_trig_fit() {
  return TrigFit{
      {0x1.921fb54436ef2p+2, -0x1.4abbce5f63211p+5, 0x1.466bc5fa6500cp+6, -0x1.32d2bd3e55934p+6, 0x1.5076469da3a25p+5, -0x1.e2c50a2af1684p+3, 0x1.e4010f5a8e8f9p+1, -0x1.3dd13c98fd649p-1},
      {0x1.ffffffff02459p-1, -0x1.3bd3cc8c07aa4p+4, 0x1.03c1ef342aa38p+6, -0x1.55d39e1715dd5p+6, 0x1.e1efdf3216450p+5, -0x1.a6795df5265d4p+4, 0x1.f333905dc4367p+2, -0x1.73f6fde455a14p+0}};
}
}  // namespace gw
