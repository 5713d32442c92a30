// The single-pass kernels on the CPU, from their own source, waves in either
// order (kernel_emulation.h): layers one after the other in the rounds of one
// plan must come out bit for bit as each of them alone in a plan of one round.
// And a wait that is not eager and one that is give up after the same time.
// Prints what differs; the exit status is 0 when nothing does.
#include "kernel_emulation.h"

#include "lamb_kernels.hip"

// The poll limit that launch_single_pass hands to its kernel; nothing else of a
// launch is looked at here.
static uint32_t launched_limit = 0;
hipError_t hipLaunchKernel(const void *, dim3, dim3, void **arguments, size_t, hipStream_t) {
    launched_limit = static_cast<const lamb_mi355x::StepArgs *>(arguments[7])->spin_limit;
    return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *, const void *, int, size_t) {
    return hipErrorNotSupported;
}

namespace {
using namespace lamb_mi355x;

struct Layer {
    std::vector<float> x, g, m, v;
    std::vector<uint16_t> copy;
    double ratio = -1.0;
    explicit Layer(int numel, uint32_t seed) {
        auto next = [&seed]() {
            seed = seed * 1664525u + 1013904223u;
            return float(int32_t(seed >> 8) - (1 << 23)) / float(1 << 23);
        };
        for (int k = 0; k < numel; ++k) {
            x.push_back(next());
            g.push_back(0.01f * next());
            m.push_back(0.01f * next());
            v.push_back(1e-4f * std::fabs(next()));
            copy.push_back(0);
        }
    }
    bool same(const Layer &o) const {
        return x == o.x && m == o.m && v == o.v && copy == o.copy && ratio == o.ratio;
    }
};

// The layer's tiles as lamb_plan_create lists them.
void add_tiles(std::vector<TileDesc> *tiles, Layer *l, int groups, int out) {
    const int32_t numel = int32_t(l->x.size());
    const int32_t n = int32_t((numel + tile_elems(groups) - 1) / tile_elems(groups));
    const int32_t blocks = (numel / 4 * 4 + kBlockElems - 1) / kBlockElems;
    const int32_t last = (numel - 1) / kBlockElems;
    for (int32_t k = 0; k < n; ++k)
        tiles->push_back(TileDesc{l->x.data(), l->g.data(), l->m.data(), l->v.data(),
                                  l->copy.data(), numel, k, n, out, -1,
                                  tile_shape(out % 2 == 0,
                                             numel % kBlockElems != 0 && last % n == k,
                                             k < blocks ? (blocks - k + n - 1) / n : 0)});
}

struct Call {
    const std::vector<TileDesc> *tiles;
    uint64_t *slots;
    uint32_t *ctl, *flags;
    double *ratios;
    bool quick;
    uint32_t spin_limit = 1u << 30;
};

template <int kAlgo, int kGroups>
void kernel_body(void *p) {
    const Call &c = *static_cast<const Call *>(p);
    StepArgs a{};
    a.beta1 = 0.9f;
    a.one_minus_beta1 = 0.1f;
    a.beta2 = 0.999f;
    a.one_minus_beta2 = 0.001f;
    a.m_scale = 10.0f;
    a.v_scale = 1000.0f;
    a.eps = 0.0f;
    a.weight_decay = 0.01f;
    a.grad_scale = 1.0f;
    a.spin_limit = c.spin_limit;
    const FinalizeArgs f{0.01, 0.0, 10.0, 1.0};
    const int32_t n = int32_t(c.tiles->size());
    if (c.quick)
        quick_kernel<kAlgo, false, kL2, kGroups>(c.tiles->data(), n, c.slots, c.ctl, c.flags, 0,
                                                 nullptr, a, f, c.ratios, nullptr, nullptr,
                                                 nullptr, nullptr);
    else
        fused_kernel<kAlgo, false, kL2, kGroups>(c.tiles->data(), n, c.slots, c.ctl, c.flags, 0,
                                                 nullptr, a, f, c.ratios, nullptr, nullptr,
                                                 nullptr, nullptr);
}

template <int kAlgo, int kGroups>
void step(std::vector<Layer> &layers, uint32_t grid, bool quick, bool last_first) {
    std::vector<TileDesc> tiles;
    for (size_t i = 0; i < layers.size(); ++i)
        add_tiles(&tiles, &layers[i], kGroups, int(i));
    std::vector<uint64_t> slots(6 * tiles.size(), kEmptySlot);
    std::vector<uint32_t> ctl(64, 0), flags(64, 0);
    std::vector<double> ratios(layers.size(), -1.0);
    Call c{&tiles, slots.data(), ctl.data(), flags.data(), ratios.data(), quick};
    std::vector<std::thread> workgroups;
    for (uint32_t w = 0; w < grid; ++w)
        workgroups.emplace_back(emulation::run_workgroup, w, grid, uint32_t(kBlock), last_first,
                                &kernel_body<kAlgo, kGroups>, &c);
    for (std::thread &t : workgroups)
        t.join();
    for (size_t i = 0; i < layers.size(); ++i)
        layers[i].ratio = ratios[i];
}

// `grid` tiles a layer and `numels.size()` rounds on `grid` workgroups.
template <int kAlgo, int kGroups>
int compare(const char *name, uint32_t grid, const std::vector<int> &numels) {
    int bad = 0;
    for (int form = 0; form < 4; ++form) {
        const bool quick = form & 1, last_first = form & 2;
        std::vector<Layer> all;
        for (size_t i = 0; i < numels.size(); ++i)
            all.emplace_back(numels[i], uint32_t(i + 1));
        step<kAlgo, kGroups>(all, grid, quick, last_first);
        for (size_t i = 0; i < numels.size(); ++i) {
            std::vector<Layer> alone;
            alone.emplace_back(numels[i], uint32_t(i + 1));
            alone.emplace_back(numels[i], 1000u);  // (keeps out_index parity: decay on)
            if (i % 2 == 1)
                std::swap(alone[0], alone[1]);
            // a plan of one round: this layer beside another one
            step<kAlgo, kGroups>(alone, 2 * grid, quick, last_first);
            if (!alone[i % 2].same(all[i])) {
                printf("%s %s, waves %s first: layer %zu of %d elements differs\n", name,
                       quick ? "quick_kernel" : "fused_kernel", last_first ? "last" : "first", i,
                       numels[i]);
                ++bad;
            }
        }
    }
    return bad;
}

// A wait that nothing ends, alone on the device: a layer of two tiles of which
// only tile `index` runs, in a plan of one round or of two. Returns its sleeps,
// or 0 when it did not give up.
uint64_t sleeps_of_a_wait(bool quick, bool one_round, uint32_t index, uint32_t limit) {
    std::vector<Layer> layers;
    layers.emplace_back(8192 + 4096, 1u);
    layers.emplace_back(8192 + 4096, 2u);
    std::vector<TileDesc> tiles;
    add_tiles(&tiles, &layers[0], 8, 0);
    if (!one_round)
        add_tiles(&tiles, &layers[1], 8, 1);
    std::vector<uint64_t> slots(6 * tiles.size(), kEmptySlot);
    std::vector<uint32_t> ctl(64, 0), flags(64, 0);
    std::vector<double> ratios(2, -1.0);
    StepArgs args{};
    args.spin_limit = limit;
    // (a plan of more than kQuickRounds rounds of one workgroup, for fused_kernel)
    const int32_t n_tiles = quick ? int32_t(tiles.size()) : 1000;
    if (launch_single_pass(StepKind{}, 8, tiles.data(), n_tiles, 2, slots.data(), ctl.data(),
                           flags.data(), false, nullptr, args, FinalizeArgs{}, nullptr, nullptr,
                           nullptr, nullptr, nullptr, nullptr) != hipSuccess)
        return 0;
    Call c{&tiles,        slots.data(), ctl.data(),     flags.data(),
           ratios.data(), quick,        launched_limit};
    uint64_t n = 0;
    std::thread([&] {
        emulation::run_workgroup(index, 2, uint32_t(kBlock), false, &kernel_body<kLamb, 8>, &c);
        n = emulation::sleeps;
    }).join();
    return ctl[kCtlFault] != 0 ? n : 0;
}

// An eager wait's polls are shorter than another wait's, by up to 1.85 times
// (0.19 to 0.23 us, 0.35): it may not give up after fewer than twice as many,
// or a step that used to wait a busy device out would be abandoned.
int check_patience() {
    constexpr uint32_t kLimit = 600;
    int bad = 0;
    auto expect = [&](const char *what, uint64_t got, uint64_t polls) {
        if (got != polls - 1) {  // (a poll that finds the limit reached does not sleep)
            printf("%s gives up after %llu polls, not %llu\n", what,
                   static_cast<unsigned long long>(got + 1),
                   static_cast<unsigned long long>(polls));
            ++bad;
        }
    };
    expect("quick_kernel, several rounds", sleeps_of_a_wait(true, false, 1, kLimit), kLimit);
    expect("fused_kernel, a member", sleeps_of_a_wait(false, true, 1, kLimit), kLimit);
    expect("quick_kernel, one round", sleeps_of_a_wait(true, true, 1, kLimit), 2 * kLimit);
    expect("quick_kernel, one round, the leader", sleeps_of_a_wait(true, true, 0, kLimit),
           2 * kLimit);
    expect("fused_kernel, an eager leader", sleeps_of_a_wait(false, true, 0, kLimit), 2 * kLimit);
    return bad;
}

}  // namespace

int main() {
    // Layers whose last 1 to 3 elements belong to threads of every wave
    // ((numel / 4) % 256), one of whole float4s and one that fills its tile.
    const std::vector<int> numels = {4 * 10 + 1,  4 * 200 + 2, 4 * (256 + 70) + 3, 4 * 255 + 1,
                                     4 * 512 + 3, 4 * 130 + 1, 3,                  4 * 128,
                                     8 * 1024,    4 * 64 + 2};
    int bad = compare<kLamb, 8>("LAMB", 1, numels);
    bad += compare<kLamb, 10>("LAMB, wide tile", 1, numels);
    bad += compare<kLars, 8>("LARS", 1, numels);
    // teams of two tiles, whose last block is in the first or the second one
    bad += compare<kLamb, 8>("LAMB, two tiles", 2,
                             {8192 + 41, 8192 + 1024 + 803, 8192 + 4097, 16384 - 3, 8192 + 1021});
    if (bad == 0)
        printf("all layers agree\n");
    const int impatient = check_patience();
    if (impatient == 0)
        printf("all waits are as patient\n");
    return bad + impatient != 0;
}
