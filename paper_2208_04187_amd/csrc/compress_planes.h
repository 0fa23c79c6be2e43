// Part of division.hip (included inside its unnamed namespace, after the kernels whose bodies it holds): compress_planes.

// ------------------------------------------------------------------ compress, small planes of several shapes in one launch

// The one-wavefront kernels of small planes over the maps of several shapes.  A launch of its own costs a shape 2-4 us of draining and filling: the
// compress side of a ResNet-18 / CIFAR step in four launches 65 us (4.4 TB/s), in one 50 (5.7).
// ALL = false: compress_strip (B = 4, 8) and compress_items under B = 4, which need 64 registers at most, as when they are alone.  ALL = true: also
// compress_rowstrip, compress_items under B = 8 and compress_lane, all at the registers of the hungriest (fp32 118 to 128, bfloat16 124 to 154): for launches of a few generations of wavefronts, where
// how many are on the machine at once matters less than that no launch waits for the one before (five shapes of a small network, compress and decompress, 43.0 ->
// 37.8 us; 60 drawn calls with compress_rowstrip in them 1119 -> 1057, with compress_lane 1152 -> 1098).
struct PlanesShape { uint32_t kind; union { StripShape strip; ItemsShape items; LaneShape lane; }; };
// kind: 100 W + B of the strips; 10 B + elements per row of an item of the items; 1 of the lane kernel
struct PlanesArgs : SharedTab {
    PlanesShape shape[kSharedShapes];
    Regions rg[kSharedShapes];
};
template <typename T, int BITS, bool ALL>
__global__ void __launch_bounds__(64) compress_planes(PlanesArgs a) {
    const SharedPlace at = shared_place(a);
    const Regions& rg = a.rg[at.shape];
    if (at.wg == 0 && threadIdx.x < 48) zero_pads(rg, static_cast<char*>(a.pk[at.map]), threadIdx.x);
    const CompPtrs pt = shared_ptrs(a, rg, at.map);
    const PlanesShape& s = a.shape[at.shape];
    const uint32_t wg = xcd_run_index(at.wg, at.n);
    if constexpr (ALL) {
        switch (s.kind) {
            case 1308: compress_rowstrip_slots<T, BITS, 13, 8>(s.strip, pt, wg); return;
            case 1304: compress_rowstrip_slots<T, BITS, 13, 4>(s.strip, pt, wg); return;
            case 1508: compress_rowstrip_slots<T, BITS, 15, 8>(s.strip, pt, wg); return;
            case 1504: compress_rowstrip_slots<T, BITS, 15, 4>(s.strip, pt, wg); return;
            case 1708: compress_rowstrip_slots<T, BITS, 17, 8>(s.strip, pt, wg); return;
            case 1704: compress_rowstrip_slots<T, BITS, 17, 4>(s.strip, pt, wg); return;
            case 2708: compress_rowstrip_slots<T, BITS, 27, 8>(s.strip, pt, wg); return;
            case 2704: compress_rowstrip_slots<T, BITS, 27, 4>(s.strip, pt, wg); return;
            case 3508: compress_rowstrip_slots<T, BITS, 35, 8>(s.strip, pt, wg); return;
            case 3504: compress_rowstrip_slots<T, BITS, 35, 4>(s.strip, pt, wg); return;
            case 5508: compress_rowstrip_slots<T, BITS, 55, 8>(s.strip, pt, wg); return;
            case 5504: compress_rowstrip_slots<T, BITS, 55, 4>(s.strip, pt, wg); return;
            case 84: compress_items_body<T, BITS, 8, 4, 8, false>(s.items, pt, wg); return;
            case 82: compress_items_body<T, BITS, 8, 2, 8, false>(s.items, pt, wg); return;
            case 1: compress_lane_body<T, BITS>(s.lane, pt, wg); return;
        }
    }
    switch (s.kind) {
        case 3208: compress_strip_body<T, BITS, 32, 8, false>(s.strip, pt, wg); break;
        case 2808: compress_strip_body<T, BITS, 28, 8, false>(s.strip, pt, wg); break;
        case 1608: compress_strip_body<T, BITS, 16, 8, false>(s.strip, pt, wg); break;
        case 1408: compress_strip_body<T, BITS, 14, 8, false>(s.strip, pt, wg); break;
        case 3204: compress_strip_body<T, BITS, 32, 4, false>(s.strip, pt, wg); break;
        case 1604: compress_strip_body<T, BITS, 16, 4, false>(s.strip, pt, wg); break;
        case 44: compress_items_body<T, BITS, 4, 4, 4, false>(s.items, pt, wg); break;
        default: compress_items_body<T, BITS, 4, 2, 4, false>(s.items, pt, wg);
    }
}
