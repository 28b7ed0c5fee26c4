"""The Box-Muller functions of the bond-force-biased moves
(csrc/soma_boxmuller.hpp), compiled for the host with g++ and compared with
long double at every one of their 2^24 arguments
(tests/helpers/boxmuller_pin.cpp).

Bounds, from the operations:
  * logarithm: one rounding of the result and one of f + tail, which is at
    most as large as the result: below 1 ulp;
  * root: a correctly rounded residual step: 0.51 ulp;
  * sine, cosine: the terms after the leading one are at most 0.58 of values in
    [0, 1]; their polynomial's last two roundings, the product with the angle
    and its sum of parts each leave at most 2^-54: 2e-16 beyond half an ulp;
  * a normal: r <= 5.9 times the sine's 2e-16, and 3 x 2^-52 for the relative
    errors of the root, the sine's last rounding and the product -- and no
    larger than the C library's.
"""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_functions_of_24_bit_arguments(tmp_path):
    exe = str(tmp_path / "boxmuller_pin")
    subprocess.check_call(["g++", "-O2", "-ffp-contract=off", "-mfma", "-std=c++17",
                           "-I", os.path.join(HERE, "..", "paper_2606_09356_amd", "csrc"),
                           os.path.join(HERE, "helpers", "boxmuller_pin.cpp"), "-o", exe])
    log, root, sine, cosine, normal, library = (
        float(v) for v in subprocess.check_output([exe], text=True).split())
    assert log < 1.0
    assert root < 0.51
    assert sine < 2e-16 and cosine < 2e-16
    assert normal <= 5.9 * 2e-16 + 3 * 2.0 ** -52
    assert normal <= library
