// Generated by gen_lskum_math.py; do not edit.
// Q(r) = (e^r - 1 - r)/r^2 on |r| <= ln2/2, degree 10, fit error 1.4e-18
constexpr double kExpQ[11] = {
    0x1.1f72fc730b4ffp-29,
    0x1.af4ddd84882fep-26,
    0x1.27e4db67b4303p-22,
    0x1.71de02375656cp-19,
    0x1.a01a01a6d7808p-16,
    0x1.a01a01abe62ddp-13,
    0x1.6c16c16c162d6p-10,
    0x1.11111111100dfp-7,
    0x1.5555555555556p-5,
    0x1.5555555555557p-3,
    0x1.0000000000000p-1};

// P(t) = erf(sqrt t)/sqrt t on [0, 1], degree 11, fit error 7.35e-18
constexpr double kErfP[12] = {
    -0x1.ac9585a44fe29p-31,
    0x1.d76af6ca49787p-27,
    -0x1.5c131500d3f88p-23,
    0x1.b981d78881a5dp-20,
    -0x1.f4ca838adb73bp-17,
    0x1.f9a2be4f731a1p-14,
    -0x1.c02db0665e53dp-11,
    0x1.565bccfa44156p-8,
    -0x1.b82ce31203772p-6,
    0x1.ce2f21a040f66p-4,
    -0x1.812746b0379c1p-2,
    0x1.20dd750429b6dp+0};

// E(u) = e^(-u) on [-1/2, 1/2], degree 12, fit error 4.98e-18
constexpr double kExpN[13] = {
    0x1.2036290a2a4e6p-29,
    -0x1.b0a38fe8033d7p-26,
    0x1.27e42df3ab7bcp-22,
    -0x1.71dcd28a56ee8p-19,
    0x1.a01a021b73430p-16,
    -0x1.a01a02780e87dp-13,
    0x1.6c16c16bf2c5dp-10,
    -0x1.11111110d2113p-7,
    0x1.55555555555e5p-5,
    -0x1.555555555574dp-3,
    0x1.0000000000000p-1,
    -0x1.fffffffffffffp-1,
    0x1.0000000000000p+0};

// W(v) = erfcx(3 (1 + v)/(1 - v)) on [-1/2, 1/3], degree 14, fit error 1.01e-17
constexpr double kErfcxW[15] = {
    0x1.57a5fe2b9b75ep-20,
    0x1.0f9a79cee3e31p-19,
    -0x1.0cb4611cc29f6p-17,
    -0x1.af2329d757293p-17,
    0x1.0cb1db32e0c9fp-14,
    0x1.7b9fc8eb630e9p-15,
    -0x1.39085a31b18abp-11,
    0x1.73101ea8fe252p-11,
    0x1.17c838fea5806p-8,
    -0x1.8fa58eb5bd68fp-6,
    0x1.258b13b0139fep-4,
    -0x1.336ffbef08cbbp-3,
    0x1.f6ff20410599bp-3,
    -0x1.4e102b9cf8512p-2,
    0x1.6e9827d229d2dp-3};

constexpr double kExpHalf = 0x1.368b2fc6f960ap-1;
constexpr double kLog2e = 0x1.71547652b82fep+0;
constexpr double kLn2Hi = 0x1.62e42fefa39efp-1;
constexpr double kLn2Lo = 0x1.abc9e3b39803fp-56;
