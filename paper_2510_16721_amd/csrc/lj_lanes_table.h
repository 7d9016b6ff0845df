// LJ lanes per atom by band size (atoms x moving images at creation): the fastest lane
// count of an FP32 LJ band stepped alone.  Written by tune_lanes.py from
// force-stage times (us per step) of LJ FCC vacancy-hop bands (the fewest lanes
// within 16 % of the fastest):
//         155 atom-images: 1:     35.0  2:     19.3  4:     13.4  8:      9.7  16:      8.3  32:      7.2
//         255 atom-images: 1:     32.2  2:     19.8  4:     14.1  8:     10.4  16:      9.0  32:      7.8
//        1275 atom-images: 1:     32.5  2:     20.3  4:     13.9  8:     10.3  16:      8.7  32:      7.6
//        2495 atom-images: 1:     23.6  2:     15.6  4:     11.8  8:      9.8  16:      8.4  32:      7.8
//        3999 atom-images: 1:     23.4  2:     15.9  4:     11.5  8:      9.3  16:      8.1  32:      8.0
//        4315 atom-images: 1:     23.6  2:     15.7  4:     11.5  8:      9.3  16:      8.6  32:      9.1
//       10235 atom-images: 1:     24.1  2:     16.1  4:     11.5  8:     10.6  16:     10.1  32:     11.2
//       18423 atom-images: 1:     24.0  2:     16.4  4:     13.4  8:     11.8  16:     13.5  32:     15.2
//       26615 atom-images: 1:     24.8  2:     16.7  4:     13.6  8:     13.5  16:     15.5  32:     19.3
//       54875 atom-images: 1:     27.8  2:     20.7  4:     19.0  8:     20.1  16:     24.0  32:     26.9
//       81915 atom-images: 1:     34.1  2:     24.8  4:     24.9  8:     26.6  16:     31.7  32:     35.4
//      147447 atom-images: 1:     41.4  2:     36.8  4:     35.8  8:     38.2  16:     47.6  32:     52.5
//      212955 atom-images: 1:     48.9  2:     49.8  4:     54.1  8:     57.7  16:     74.8  32:     85.1
//      487775 atom-images: 1:     91.6  2:     94.9  4:    103.3  8:    112.2  16:    144.6  32:    161.2
//     2146210 atom-images: 1:    349.0  2:    382.0  4:    419.5  8:    449.6  16:    578.8  32:    639.8
#ifndef CFNEB_LJ_LANES_TABLE_H
#define CFNEB_LJ_LANES_TABLE_H

struct LjLanesEntry {
    long long max_atom_images;
    int lanes;
};
static const LjLanesEntry kLjLanesTable[] = {
    {4153LL, 16},
    {6645LL, 8},
    {38216LL, 4},
    {109900LL, 2},
    {9223372036854775807LL, 1},
};

#endif
