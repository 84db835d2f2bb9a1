// mds_coeffs.h -- generated by gen_coeffs.py; do not edit by hand.
// Coefficients are listed from the constant term upwards (Horner order reversed).
#pragma once

#include <hip/hip_runtime.h>

namespace mds {

// erfcx(z) ~ P(z)/Q(z) on [0, 27.5] (FP64); worst relative error 6.44e-16 with FP64 coefficients
constexpr double kErfcxZmax64 = 27.5;
constexpr double kErfcxP64[10] = {
    0x1.0000000000000p+0,
    0x1.1880e4819767ap+1,
    0x1.30163d40a64cfp+1,
    0x1.a2dd47a01da1dp+0,
    0x1.9000926828a37p-1,
    0x1.11844cb5dc3f3p-2,
    0x1.0bce512a10e4bp-4,
    0x1.6b4c6c248fedap-7,
    0x1.3829d5e0cd66dp-10,
    0x1.06a75665f1eb1p-14};

constexpr double kErfcxQ64[11] = {
    0x1.0000000000000p+0,
    0x1.a8ef9f03ac412p+1,
    0x1.47c9b49ebda04p+2,
    0x1.3642e5643bbc2p+2,
    0x1.9044d29f7bfe4p+1,
    0x1.710e5dece4ebdp+0,
    0x1.eeccec0584cb5p-2,
    0x1.deff0b1ef7daap-4,
    0x1.42dfcb4a99972p-6,
    0x1.14a5caee6bd63p-9,
    0x1.d18a9f6773061p-14};

// erfcx(z) ~ P(z)/Q(z) on [0, 10.25] (FP32); worst relative error 2.36e-07 with FP32 coefficients
constexpr float kErfcxZmax32 = 10.25f;
constexpr float kErfcxP32[5] = {
    0x1.0000000000000p+0f,
    0x1.3d46aa0000000p+0f,
    0x1.7713f20000000p-1f,
    0x1.d65dcc0000000p-3f,
    0x1.0d69900000000p-5f};

constexpr float kErfcxQ32[6] = {
    0x1.0000000000000p+0f,
    0x1.2f12140000000p+1f,
    0x1.33bf320000000p+1f,
    0x1.53c1b80000000p+0f,
    0x1.a0e0ba0000000p-2f,
    0x1.dd83f00000000p-5f};

// erfcx(z) ~ P(z)/Q(z) on [2.1, 6.6] (FP64, t = z sqrt 2 >= 3.0 up to rounding); worst relative error 6.55e-16 with FP64 coefficients
constexpr double kFarT = 3.0;
constexpr double kErfcxFarZmin64 = 2.1;
constexpr double kErfcxFarZmax64 = 6.6;
constexpr double kErfcxFarP64[7] = {
    0x1.0000936f31967p+0,
    0x1.ce6d5ac365e72p+0,
    0x1.967a937c125bcp+0,
    0x1.b2199cbf96026p-1,
    0x1.294354e849ffep-2,
    0x1.f5988efb33986p-5,
    0x1.bbb9f6d005233p-8};

constexpr double kErfcxFarQ64[8] = {
    0x1.0000000000000p+0,
    0x1.77a77992f528ep+1,
    0x1.f317535e25d32p+1,
    0x1.8863ea11bba99p+1,
    0x1.8e9a72ab7a51cp+0,
    0x1.0a83be522e087p-1,
    0x1.bc87206f17fe2p-4,
    0x1.893e076c0501fp-7};

// erfcx(t/sqrt 2)/2 ~ P(t)/Q(t) on [0, 9.0] (FP64); worst relative error 6.21e-16 with FP64 coefficients
constexpr double kNearP64[9] = {
    0x1.0000000000000p-1,
    0x1.540ee0c705426p-1,
    0x1.c2582417095a7p-2,
    0x1.7680023cd4bd4p-3,
    0x1.a61e8d4a7e6b0p-5,
    0x1.484d931b82bedp-7,
    0x1.57e8088229545p-10,
    0x1.bd41e1e8e3bb7p-14,
    0x1.133233092929bp-18};

constexpr double kNearQ64[10] = {
    0x1.0000000000000p+0,
    0x1.10288532d37adp+1,
    0x1.09bca9dbbc296p+1,
    0x1.399b93a17a613p+0,
    0x1.ee8ac3bcbfb3dp-2,
    0x1.0f3753b4199cfp-3,
    0x1.9fd3aa0134ecfp-6,
    0x1.b05eb4dc521f4p-9,
    0x1.17061008b501fp-12,
    0x1.58e83abf6f9e2p-17};

// 2^f on |f| <= 1/2, degree 11; worst relative error 2.12e-16
constexpr double kExp2C64[12] = {
    0x1.0000000000000p+0,
    0x1.62e42fefa39efp-1,
    0x1.ebfbdff82c598p-3,
    0x1.c6b08d704a0c2p-5,
    0x1.3b2ab6fba1ddap-7,
    0x1.5d87fe78a5276p-10,
    0x1.430913096fd9fp-13,
    0x1.ffcbfc670dcd4p-17,
    0x1.62bfd47773353p-20,
    0x1.b524fae627834p-24,
    0x1.e6063f7217bc6p-28,
    0x1.e9d3fe3952179p-32};

// exp(x) = 2^k exp(r), x = k ln2 + r, |r| <= ln2/2; ln2 = head + tail with
// head on 33 significant bits so that k*head is exact for |k| < 2^20
constexpr double kLn2Head = 0x1.62e42fef00000p-1;
constexpr double kLn2Tail = 0x1.473de6af278edp-34;
constexpr double kLog2e = 0x1.71547652b82fep+0;
constexpr double kLog2eTail = 0x1.777d0ffda0d24p-56;  // log2(e) - kLog2e
// Taylor polynomial of exp(r), degree 12; worst relative error 3.14e-16
constexpr double kExpC64[13] = {
    0x1.0000000000000p+0,
    0x1.0000000000000p+0,
    0x1.0000000000000p-1,
    0x1.5555555555555p-3,
    0x1.5555555555555p-5,
    0x1.1111111111111p-7,
    0x1.6c16c16c16c17p-10,
    0x1.a01a01a01a01ap-13,
    0x1.a01a01a01a01ap-16,
    0x1.71de3a556c734p-19,
    0x1.27e4fb7789f5cp-22,
    0x1.ae64567f544e4p-26,
    0x1.1eed8eff8d898p-29};

// A(v) = atanh(sqrt v)/sqrt v on [0, 1/9], so that log1p(-q) = -2 s A(s^2),
// s = q/(2-q); FP64 degree 11: worst relative error 2.20e-16; FP32 degree 5: 5.96e-08
constexpr double kAtanhA64[12] = {
    0x1.0000000000000p+0,
    0x1.5555555555557p-2,
    0x1.9999999999495p-3,
    0x1.24924924c6d06p-3,
    0x1.c71c71a3ae0a8p-4,
    0x1.745d1e4e8048ep-4,
    0x1.3b12cf4f56673p-4,
    0x1.1123a50c5a1ecp-4,
    0x1.dfdb8efa1c534p-5,
    0x1.c19a2aecea0b3p-5,
    0x1.1deab3109560fp-5,
    0x1.51ae1ac364a94p-4};

constexpr float kAtanhA32[6] = {
    0x1.0000000000000p+0f,
    0x1.55555a0000000p-2f,
    0x1.9996380000000p-3f,
    0x1.2512280000000p-3f,
    0x1.b63e160000000p-4f,
    0x1.f396560000000p-4f};

}  // namespace mds
