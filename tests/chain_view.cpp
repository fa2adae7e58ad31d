// What the host works out for the chains of a loaded ensemble (csrc/chain.h), for tests on a machine without a GPU.
#include "chain.cpp"

using namespace ens;

extern "C" {

int chain_steps(ens_handle* h, int member) { return h->chains.empty() ? 0 : (int)h->chains[member].steps.size(); }

int chain_cap(ens_handle* h, int member) { return h->chains.empty() ? 0 : h->chains[member].cap; }

// How many wavefronts share the K of a member's convolution with `K` and `cout` in a program of up to 1 << z images, as a power of two; -1: none such.
int chain_split(ens_handle* h, int member, int K, int cout, int z) {
    for (const ChainStep& s : h->chains[member].steps)
        if (s.kind <= CH_CONV_PRE && s.K == K && s.cout == cout) return s.choice[z] >> 8 & 255;
    return -1;
}

// The tiles of a member's phases beside those of each convolution by itself: 1: K in other parts; 2: the phase takes longer; 4: more units than a step counts;
// 8: a phase of one step does not take what its step takes.  `better`: phases that take less, `most`: the most units of a step.
int chain_tiles_wrong(ens_handle* h, int member, int* better, int* most) {
    int wrong = 0;
    *better = *most = 0;
    const std::vector<ChainStep>& all = h->chains[member].steps;
    for (size_t i = 0; i < all.size();) {
        const int count = all[i].phase_steps & 255;
        for (int z = 0; z < CHAIN_SIZES; z++) {
            std::vector<ChainStep> chosen(all.begin() + i, all.begin() + i + count), own = chosen;
            for (int j = 0; j < count; j++) {
                ChainStep& s = own[j];
                const double n = units(s, 1 << z, s.choice[z]);
                if (n > 65535.0 || (int)((unsigned)s.choice[z] >> 16) != (int)n) wrong |= 4;
                *most = std::max(*most, (int)n);
                if (s.kind <= CH_CONV_PRE) s.choice[z] = own_tiles(s, 1 << z);
                if (s.kind <= CH_CONV_PRE && (s.choice[z] >> 8 & 255) != (chosen[j].choice[z] >> 8 & 255)) wrong |= 1;
                const double one = phase_us(&s, 1, 1 << z, z), step = step_us(s, 1 << z, z);
                if (std::fabs(one - step) > 1e-9 * step) wrong |= 8;
            }
            const double us = phase_us(chosen.data(), count, 1 << z, z), by_own = phase_us(own.data(), count, 1 << z, z);
            if (us > by_own + 1e-9) wrong |= 2;
            *better += us < by_own - 1e-9;
        }
        i += count;
    }
    return wrong;
}

// What a group leaves that gave up waiting.
void chain_gave_up(ens_handle* h) { h->flag[CHAIN_FAILED_WORD] = 1; }

// The weights that the convolutions of a member ask for, with every tile that is chosen for some number of images: the number of
// fragments of which a lane lies outside the layer's weights, and of those that are asked for and do not exist (`none`).
int chain_weights_outside(ens_handle* h, int member, int* none) {
    int outside = 0;
    *none = 0;
    for (const ChainStep& s : h->chains[member].steps) {
        if (s.kind > CH_CONV_PRE) continue;
        const int chunks = (s.K + 63) / 64;
        bool sides[3] = {false, false, false};
        for (int z = 0; z < CHAIN_SIZES; z++) sides[s.choice[z] & 255] = true;
        for (int side = 1; side <= 2; side++)
            for (int cs = 0; sides[side] && cs < s.ctiles[side - 1]; cs++)
                for (int i = 0; i < side; i++)
                    for (int m = 0; m < chunks; m++)
                        for (int st = 0; st < 4; st++) {
                            const unsigned at = chain_weight_lane(cs, side, i, s.ctiles[0], 63);
                            const size_t block = (size_t)(((cs * side + i) * chunks + m) * 4 + st) * 1024;
                            if (at >= 0x80000000u) (*none)++;    // zeros
                            else outside += block + at + 16 > (size_t)s.wsize;
                        }
    }
    return outside;
}

}
