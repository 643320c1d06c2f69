// Whether a module runs level by level, its steps sharing launches, or branch by branch (api.hip).  Plain constant expressions, so that the same lines run
// in the library and in a test on the host.
#pragma once

namespace dr {

// What a module's convolutions are: all of them, those that the kernels for small layers take, larger ones that may share a launch; and of the two branches
// with the longest contractions outside the kernels that share launches (channels not in eights, filters in KCRS order, ...) how long these are, added up
struct ModuleLayers { int all, small, big; long longest, second; };

// At least two convolutions that can share, and with the branches wanted on streams:
// bf16: unless two branches have layers that share nothing, one at least two fifths as long as the other.  The layers of a depth lie side by side in one launch, each
// with its share of the compute units (as graphs, streams and levels: the original GoogLeNet on 12 images 487 and 360 us, on 40 746 and 581, on 128 1494 and
// 1367; the fused one 297 and 260, 492 and 414, 1042 and 968; on six and fewer, where every layer is small, both went by levels), and a layer that shares nothing
// runs behind them (eager, 4c on 12 images: a 5x5 on 12 channels 111 and 53 us, a 3x3 on 92 in 4a 113 and 85, a 5x5 beyond the chunk table 115 and 73).  Two of
// those are better off side by side, the more the closer they are: 5b with a 3x3 on 188 channels and a 5x5 on 44 195 and 235, 4e with 156 and 28 172 and 198,
// 4c on 484 channels, four such branches, 125 and 188; in 4a with 92 and 12 (828 and 300 long) the two ways take the same time, 0.93 to 1.11 on 4 to 100 images.
// fp32: only where every convolution can share, and most of them in the small-layer kernel: a level is a barrier between the branches, and larger layers, which
// share a launch one tile after the other, fill the device better on streams (4c on 64 images, one small layer of six: 203 against 237), while a large layer
// among small ones does not (slim 5a on 64 images, a 5x5 of 392 tiles beside three small layers: 113 against 95, as graphs).
constexpr bool module_by_levels(const ModuleLayers& m, bool bf16, bool streams)
{
    if (m.small + m.big < 2) return false;
    if (!streams) return true;
    return bf16 ? m.second == 0 || 5 * m.second < 2 * m.longest : m.small + m.big == m.all && 2 * m.small > m.all;
}

}  // namespace dr
