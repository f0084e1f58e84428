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

// Runs in small blocks, 32 channels wide where 64 would leave the chip half
// empty, and k_conv_fwd_lds where its wider blocks fill it.  Resident are 768
// blocks of 128 channels (three per CU), 1280 of k_conv_fwd_run<64> (five).
// Every output width from 32 to 384, 64 to 768 input channels, 64 to 2^20
// pixels (us, k_conv_fwd_lds / 64 wide / 32 wide):
//   128 outputs and multiples: 256 inputs, 2^18 pixels 255 / 391 / 794, 98304
//   100 / 147 / 245, 65536 78 / 80 / 121; 128 inputs, 2^18 pixels 148 / 187 / 353;
//   384 inputs, 65536 pixels 111 / 119 / 209; 256 -> 256 inputs, 16384 pixels 67 /
//   55 / 58, 1024 pixels 65 / 45 / 36.  Short sums lose more by a last round that
//   is nearly empty than they gain by width: 64 -> 256, 65536 pixels (1024 blocks)
//   1.29 times 64 wide.
//   FP32 outputs alone, which k_conv_fwd_lds writes faster than BF16: 128 inputs,
//   65536 pixels 38 and 41, 384 inputs, 50176 pixels 97 and 107.
//   64 and odd multiples: 512 inputs, 65536 pixels 120 / 144 / 139, 192 inputs, 2^18
//   pixels 149 / 156 / 290; 128 inputs, 65536 pixels 6 % slower than 64 wide.
//   32 and odd multiples: 96 inputs, 2^20 pixels 193 / - / 195; below 1024 blocks
//   k_conv_fwd_run is up to 1.4 times as fast.
inline ConvForm conv_form(int B, int H, int W, int cin, int cout, bool f32)
{
    if (cin == 32 && conv_tiles_pay(B, H, W, cout)) return kConvTile;
    const long long runs = ((long long)B * H * W + 127) / 128;
    if (cout % 64 != 0) return runs * (cout / 32) > 1024 ? kConvLds : kConvRun32;
    const long long narrow = runs * (cout / 64);
    bool lds;
    if (cout % 128 == 0) {
        const long long blocks = runs * (cout / 128), rounds = (blocks + 767) / 768;
        const bool filled = 4 * blocks > 3 * 768 * rounds;
        const int least = !f32 || cin < 128 ? (cin > 256 ? 512 : 640) : (cin > 256 ? 384 : 512);
        lds = blocks >= least && (cin >= 128 || filled);
    } else {
        lds = narrow > 1280 || (cin >= 224 && narrow >= 512);
    }
    return lds ? kConvLds : narrow > 384 ? kConvRun64 : kConvRun32;
}

}  // namespace mdfnn
