// nn_rules.h -- which kernel a 3x3 convolution takes (nn_kernels.hip), by its sizes.
#pragma once

namespace mdfnn {

enum ConvForm {
    kConvTile,      // k_conv_fwd_tile: 16 x 16 pixels, 32 input channels
    kConvRun32,     // k_conv_fwd_run: 128 pixels by 32 output channels
    kConvRun64,     // the same by 64
    kConvLds        // k_conv_fwd_lds: 128 pixels by 128, 64 or 32
};

// Pixel tiles where they cover the images with little waste, or are few enough
// for one round of the chip, whose length then counts and not the padding:
// 16 x 256 x 256 pixels, 32 -> 32 channels 66 us against 130 in runs of 128
// pixels; but 16 x 9 x 1000 (1.8 times padded, 1008 tiles) 21 against 19.
inline bool conv_tiles_pay(int B, int H, int W, int cout)
{
    const long long tiles = (long long)B * ((H + 15) / 16) * ((W + 15) / 16);
    return tiles * (cout / 32) <= 512 || tiles * 256 * 5 <= 8LL * B * H * W;
}

// What a call asks of the outputs: a bias, the mask of a data gradient, FP32
// alone.
struct ConvOuts {
    bool bias, mask, f32;
};

// Runs in small blocks, 32 channels wide where 64 would leave the chip half
// empty, and k_conv_fwd_lds where its wider blocks win: in rounds of resident
// blocks (768 of 128 channels, three per CU; 1280 of k_conv_fwd_run<64>, five),
// in many blocks, or in long sums.  It writes one channel at a time: a mask, and a
// bias under short sums, cost it more.  Every output width of 32 to 384, 32 to 768
// inputs, 2^10 to 2^20 pixels (us, k_conv_fwd_lds / 64 wide / 32 wide, with bias and
// with a mask):
//   128 outputs, 256 inputs, 2^18 pixels 274 / 392 / 790 and 283 / 390 / 824, 98304 (one
//   round and two) 104 / 153 / 244 and 106 / 150 / 254, 65536 79 / 81 / 123 and 80 / 81 /
//   127; 128 inputs, 131072 pixels 92 / 93 / 149 and 96 / 92 / 166; 64 inputs, 2^18
//   pixels 109 / 102 / 128 and 115 / 99 / 145; 384 inputs, 65536 pixels 111 / 125 / 212
//   and 112 / 126 / 216; 256 outputs, 256 inputs, 16384 pixels 67 / 55 / 58 and 68 / 53 /
//   58; without bias, 384 inputs, 16 x 56 x 56 pixels 99 / 107; FP32 alone without bias,
//   128 inputs, 65536 pixels 38 / 41, 64 -> 64, 2^18 pixels 48 / 51.
//   64 outputs, 192 inputs, 2^18 pixels 150 / 157 / 289 and 156 / 157 / 304; 64 inputs 57 /
//   57 / 67 and 65 / 54 / 73; 512 inputs, 65536 pixels 120 / 143 / 140 and 123 / 142 / 141.
//   32 outputs, 96 inputs (64 + 32), 2^18 pixels 62 / - / 67 and 65 / - / 68; 128 inputs,
//   2^20 pixels 329 / - / 353 and 350 / - / 403, 131072 pixels 42 / - / 37 and 44 / - /
//   37.
inline ConvForm conv_form(int B, int H, int W, int cin, int cout, ConvOuts o)
{
    if (cin == 32 && conv_tiles_pay(B, H, W, cout)) return kConvTile;
    const long long runs = ((long long)B * H * W + 127) / 128;
    if (cout % 64 != 0) return cin >= 96 && runs * (cout / 32) >= 2048 ? kConvLds : kConvRun32;
    const long long narrow = runs * (cout / 64), blocks = narrow / 2;
    bool lds;
    if (cout % 128 == 0) {
        const bool fewer = (blocks + 767) / 768 < (narrow + 1279) / 1280;
        if (cin < 96) {
            lds = fewer && !o.mask && (blocks <= 768 || !o.bias);
        } else {
            long long least = 1280;
            if (cin >= 192) least = o.mask && cin < 256 ? 1024 : 640;
            if (cin > 256 || (cin >= 128 && !o.bias && !o.mask)) least = 512;
            if (cin > 256 && !o.bias && !o.mask) least = 384;
            lds = fewer || blocks >= least;
        }
    } else {
        lds = ((cin >= 128 || (o.f32 && !o.bias)) && !o.mask && narrow > 1280) || (cin >= 288 && narrow > 384 && narrow <= 512);
    }
    return lds ? kConvLds : narrow > 384 ? kConvRun64 : kConvRun32;
}

}  // namespace mdfnn
